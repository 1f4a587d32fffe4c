// The 128 x 128 x 64 form of the four-wavefront kernel with an assembly k loop (gemm_w4a.hip
// describes the structure): wavefront tile 64 x 64 = 4 x 4 accumulators, one workgroup per
// compute unit.  It is for problems of at most one 128 x 128 tile per compute unit, where the
// phase-alternating kernel of that tile runs alone on its compute unit and its k step (a
// quarter of a microsecond of MFMAs) is shorter than the time a copy takes to arrive from L2,
// which its two or three buffers cannot cover.  Here the LDS is a ring of five stages (160 KB:
// copies run four k steps ahead), and a wavefront issues its 32 MFMAs of a k step back to
// back, with the 24 LDS reads and 8 copies of the step in their shadow and one barrier
// (gemm_w4a128_loop.inc, written by gen_w4a128_loop.py).
//
// C is read, added and stored behind the loop.  A k tail (K % 64
// != 0) is one unpipelined step through registers after the loop.  With a split k loop (skinny
// f32 problems) a workgroup multiplies a part of the k steps of its tile and adds the result to
// C atomically instead.  Requirements as for the other tuned kernels: A, B 16-byte aligned;
// lda, ldb, K, N multiples of 8.  Rows >= M / columns >= N are fetched from clamped addresses
// and never stored.
#include "gemm_device.h"
#include "../../include/gemm_f16.h"
#include "gemm_w4a128_loop.inc"

namespace {

using namespace gemm_dev;

constexpr int SBM = 128, SBN = 128;
constexpr int A_BUF = SBM * BK * 2;          // 16 KB
constexpr int B_BUF = BK * SBN * 2;          // 16 KB
constexpr int STAGE = A_BUF + B_BUF;         // a stage of the ring: A, then B
constexpr int STAGES = 5;                    // copies run STAGES - 1 k steps ahead
constexpr int W4A128_LDS = STAGES * STAGE;   // 160 KB
constexpr int B_ROW = SBN * 2;               // bytes per k row of a B stage
constexpr int NCOPY = 4;                     // copies per wavefront per A (or B) stage

// A wave-uniform pointer, said so that it is held in scalar registers (the copies take their
// base address from a scalar register pair).
__device__ __forceinline__ const char* uniform_ptr128(const void* ptr)
{
    const uint64_t v = (uint64_t)(uintptr_t)ptr;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return (const char*)(uintptr_t)(((uint64_t)hi << 32) | lo);
}

template <typename CT, bool SPLIT>
__global__ __launch_bounds__(256) void gemm_w4a128_kernel(const TiledParams params)
{
    __shared__ __attribute__((aligned(1024))) char smem[W4A128_LDS];
    const uint32_t smem_base = (uint32_t)(uintptr_t)(lds_ptr_t)smem;

    // The split form reads its parameters all at once: in the order of their use it waited for scalar
    // loads four times in a row, 0.45 us of a call ((952,8,7376) f32 13.2 us, at once 12.3).
    TiledParams p = params;
    if constexpr (SPLIT)
        asm volatile("" : "+s"(p.M), "+s"(p.N), "+s"(p.K), "+s"(p.A), "+s"(p.lda), "+s"(p.B), "+s"(p.ldb), "+s"(p.C), "+s"(p.ldc),
                          "+s"(p.tiles_m), "+s"(p.tiles_n), "+s"(p.group_m), "+s"(p.num_xcd), "+s"(p.k_split), "+s"(p.parts_apart));

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm_base = (wave >> 1) * 64, wn_base = (wave & 1) * 64;

    // Split k (f32 C, no fused epilogue, few tiles and a long k loop: every compute unit should
    // stream operands): a workgroup takes one tile and one part of the k steps, and
    // adds its sums to C with atomic f32 additions -- C holds the old C already, the order of the
    // additions is not fixed.  Which XCD takes what: `parts_apart`.  K_len = this workgroup's part of K (all of it without a split).
    constexpr bool split = SPLIT;
    const int num_tiles = p.tiles_m * p.tiles_n;
    int part = 0, tile_m, tile_n;
    if (!split) tile_of_block(p, blockIdx.x, tile_m, tile_n);
    else {
        const int l = p.parts_apart ? xcd_slice(num_tiles * p.k_split, p.num_xcd, blockIdx.x) : (int)blockIdx.x;
        part = l / num_tiles;
        const int t = l - part * num_tiles;
        tile_in_order(p, p.parts_apart ? t : xcd_slice(num_tiles, p.num_xcd, t), tile_m, tile_n);
    }
    const int m0 = tile_m * SBM, n0 = tile_n * SBN;
    const bool edge = (m0 + SBM > p.M) || (n0 + SBN > p.N);

    const int k_steps = p.K / BK + (p.K % BK != 0);
    const int steps_per_part = split ? (k_steps + p.k_split - 1) / p.k_split : 0;
    if (split && part * steps_per_part >= k_steps) return;     // more parts than k steps: nothing to add
    const int k_begin = part * steps_per_part * BK;            // < K
    const int K_len = split ? (p.K - k_begin < steps_per_part * BK ? p.K - k_begin : steps_per_part * BK) : p.K;
    const int kt_full = K_len / BK;

    // ---- copy plan ------------------------------------------------------------------
    // A stage = 16 wave-wide copies of 8 rows x 128 B; wavefront w takes copies q = w + 4t.
    // Lane i writes (row 8q + i/8, chunk position i%8), which holds logical chunk position
    // ^ ((row/2)%8) = 4 (w%2) + i/16, the same for every t.
    const half_t* const a_tile = p.A + (int64_t)m0 * p.lda + k_begin;
    const half_t* const b_tile = p.B + (int64_t)k_begin * p.ldb + n0;
    const int a_chunk = (lane & 7) ^ (4 * (wave & 1) + (lane >> 4));
    uint32_t a_off[NCOPY];
#pragma unroll
    for (int t = 0; t < NCOPY; t++) {
        int row = 8 * (wave + 4 * t) + (lane >> 3);
        row = (m0 + row < p.M) ? row : p.M - 1 - m0;                 // clamp: loaded, never stored
        a_off[t] = ((uint32_t)row * (uint32_t)p.lda + 8 * a_chunk) * 2;
    }
    // B stage = 16 copies of 4 k rows x 256 B; copy q = w + 4t covers k rows 4q .. 4q+3.
    // Lane i writes (k row 4q + i/16, chunk position i%16), which holds logical chunk position
    // ^ swz(k row), swz = 4*(row%4) + 2*((row/8)%2) = 4 (i/16) + 2 ((w/2)%2), the same for every t.
    uint32_t b_off[NCOPY];
    const int b_krow0 = 4 * wave + (lane >> 4);                       // k row of copy t: b_krow0 + 16t
    {
        const int swz = ((lane >> 4) << 2) | (((wave >> 1) & 1) << 1);
        int col = 8 * ((lane & 15) ^ swz);
        if (n0 + col + 8 > p.N) col = 0;                              // clamp: loaded, never stored
#pragma unroll
        for (int t = 0; t < NCOPY; t++) b_off[t] = ((uint32_t)(b_krow0 + 16 * t) * (uint32_t)p.ldb + col) * 2;
    }
    const uint32_t lds_wave = smem_base + 1024 * wave;

    // ---- fragment read addresses ------------------------------------------------------
    // A operand of the 16x16x32 MFMA: lane l holds tile row l%16 of its 16-row block, k =
    // 8*(l/16)..+7 of the 32-wide slice s -> logical chunk 4s + l/16, stored at chunk ^ ((row/2)%8).
    uint32_t a_rd[2];
    {
        const uint32_t row_off = (uint32_t)(wm_base + (lane & 15)) * (BK * 2);
        const int sw = (lane & 15) >> 1;
#pragma unroll
        for (int s = 0; s < 2; s++)
            a_rd[s] = smem_base + row_off + (uint32_t)(((4 * s + (lane >> 4)) ^ sw) * 16);
    }
    // B operand: lane l holds column l%16, the same k.  One transposing read serves 16 lanes:
    // lanes 4r..4r+3 of a 16-lane block point at 16 consecutive columns of k row r and lane i
    // receives column i of rows 0..3.  Block b covers k 8b..8b+7 of the slice in two reads.
    uint32_t b_rd[4];
    {
        const int blk = lane >> 4, j = lane & 15;
        const uint32_t row_off = (uint32_t)(8 * blk + (j >> 2)) * B_ROW;
        const int swz = ((j >> 2) << 2) | ((blk & 1) << 1);           // of k rows 8b + j/4 (+4, +32)
#pragma unroll
        for (int fn = 0; fn < 4; fn++) {
            const int chunk = 2 * ((wn_base >> 4) + fn) + ((j & 3) >> 1);   // 16-byte chunk of columns 4(j%4)..+3
            b_rd[fn] = smem_base + A_BUF + row_off + (uint32_t)((chunk ^ swz) * 16 + 8 * (j & 1));
        }
    }

    // ---- C: requested behind the loop, by whole row segments of the wavefront's 64 columns, 16 bytes a lane.
    // (Before the loop, in the order of copies and waits, C kept the first k steps waiting for
    // longer than it saved behind the loop; and in the accumulators' own layout, consecutive lanes in different rows,
    // the memory pipeline takes a lane a clock, 1.7 us each way.  2048^2, K = 64 / 1024 / 4096: f32 12.7 / 19.4 /
    // 40.0 -> 11.0 / 17.4 / 37.5 us, f16 9.0 / 16.1 / 36.6 -> 7.8 / 14.8 / 35.5.)
    CT* const Cbase = (CT*)p.C;
    const int c_lrow = lane & 15, c_lcol = 4 * (lane >> 4);           // transposed 16 x 16 blocks: register r of lane l is row l%16, column 4*(l/16) + r
    const int c_row0 = m0 + wm_base, c_col0 = n0 + wn_base;
    constexpr int VEC = 16 / (int)sizeof(CT), TPR = 64 / VEC, RPP = 64 / TPR, PASSES = 64 / RPP;   // elements a lane; lanes a row; rows a pass; passes
    typedef CT ctv __attribute__((ext_vector_type(VEC), aligned(sizeof(CT))));
    const int r_row = lane / TPR, r_x = VEC * (lane % TPR);
    const bool r_col_in = c_col0 + r_x < p.N;                         // N is a multiple of 8: all of the lane's columns or none
    const uint32_t r_voff = ((uint32_t)r_row * (uint32_t)p.ldc + (uint32_t)r_x) * (uint32_t)sizeof(CT);
    auto r_ok = [&](int ps) -> bool { return !edge || (r_col_in && c_row0 + RPP * ps + r_row < p.M); };
    auto r_at = [&](int ps) -> ctv* { return reinterpret_cast<ctv*>(reinterpret_cast<char*>(Cbase + (int64_t)(c_row0 + RPP * ps) * p.ldc + c_col0) + r_voff); };
    ctv rin[PASSES];
    auto fetch_rows = [&]() {
#pragma unroll
        for (int ps = 0; ps < PASSES; ps++) { rin[ps] = ctv{}; if (r_ok(ps)) rin[ps] = *r_at(ps); }
    };
    floatx4 acc[4][4];
    if (kt_full > 0) {
        // k steps 0..3 into stages 0..3 (a k step beyond the last one: k step 0 once more, which
        // nobody reads; the loop's waits count on 8 copies per stage); the loop copies from k
        // step 4 on.  Only k step 0 is waited for here: the wait
        // in the middle of k step j leaves the 20 copies behind those of step j + 1 in flight,
        // which holds from j = 0 on with steps 2, 3 and half of 4 behind step 1.
#pragma unroll
        for (int s = 0; s < STAGES - 1; s++) {
            const int ks = s < kt_full ? s : 0;
            const char* const a_src = uniform_ptr128(a_tile + (int64_t)ks * BK);
            const char* const b_src = uniform_ptr128(b_tile + (int64_t)ks * BK * p.ldb);
#pragma unroll
            for (int t = 0; t < NCOPY; t++) async_copy16(a_src, a_off[t], lds_wave + s * STAGE + 4096 * t);
#pragma unroll
            for (int t = 0; t < NCOPY; t++) async_copy16(b_src, b_off[t], lds_wave + s * STAGE + A_BUF + 4096 * t);
        }
        asm volatile("s_waitcnt vmcnt(24)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");

        const uint64_t a_base = (uint64_t)(uintptr_t)a_tile, b_base = (uint64_t)(uintptr_t)b_tile;
        const uint32_t b_step = (uint32_t)BK * (uint32_t)p.ldb * 2u;                // bytes per k step of B (ldb <= 2^22)
        const uint64_t a_ptr = a_base + (STAGES - 1) * BK * 2, b_ptr = b_base + (STAGES - 1) * (uint64_t)b_step;
        const uint32_t a_base_lo = __builtin_amdgcn_readfirstlane((uint32_t)a_base), a_base_hi = __builtin_amdgcn_readfirstlane((uint32_t)(a_base >> 32));
        const uint32_t b_base_lo = __builtin_amdgcn_readfirstlane((uint32_t)b_base), b_base_hi = __builtin_amdgcn_readfirstlane((uint32_t)(b_base >> 32));
        const uint32_t a_ptr_lo = __builtin_amdgcn_readfirstlane((uint32_t)a_ptr), a_ptr_hi = __builtin_amdgcn_readfirstlane((uint32_t)(a_ptr >> 32));
        const uint32_t b_ptr_lo = __builtin_amdgcn_readfirstlane((uint32_t)b_ptr), b_ptr_hi = __builtin_amdgcn_readfirstlane((uint32_t)(b_ptr >> 32));
        asm volatile(W4A128_LOOP_ASM : W4A128_LOOP_OUTPUTS(acc) : W4A128_LOOP_INPUTS : W4A128_LOOP_CLOBBERS);
    } else {
#pragma unroll
        for (int fm = 0; fm < 4; fm++)
#pragma unroll
            for (int fn = 0; fn < 4; fn++) acc[fm][fn] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
    }

    if constexpr (!SPLIT) fetch_rows();
    // ---- k tail: one unpipelined step through registers, zero beyond K ------------------
    if (K_len % BK != 0) {
        __builtin_amdgcn_s_barrier();                // every wavefront is out of the loop and its copies have landed: stage 0 is free
        const int k0 = kt_full * BK, krem = K_len - k0;
        const char* a_src = (const char*)(a_tile + k0);
        const char* b_src = (const char*)(b_tile + (int64_t)k0 * p.ldb);
#pragma unroll
        for (int t = 0; t < NCOPY; t++) {
            uintx4 va = {0u, 0u, 0u, 0u}, vb = {0u, 0u, 0u, 0u};
            if (8 * a_chunk < krem) va = *reinterpret_cast<const uintx4*>(a_src + a_off[t]);
            if (b_krow0 + 16 * t < krem) vb = *reinterpret_cast<const uintx4*>(b_src + b_off[t]);
            *(__attribute__((address_space(3))) uintx4*)(uintptr_t)(lds_wave + 4096 * t + 16 * lane) = va;
            *(__attribute__((address_space(3))) uintx4*)(uintptr_t)(lds_wave + A_BUF + 4096 * t + 16 * lane) = vb;
        }
        __syncthreads();
#pragma unroll
        for (int s = 0; s < 2; s++) {
            half8 fa[4], fb[4];
#pragma unroll
            for (int fn = 0; fn < 4; fn++) {
                const uint32_t addr = b_rd[fn] + s * 32 * B_ROW;
                fb[fn] = __builtin_shufflevector(lds_read_tr16(addr), lds_read_tr16(addr + 4 * B_ROW), 0, 1, 2, 3, 4, 5, 6, 7);
            }
#pragma unroll
            for (int fm = 0; fm < 4; fm++) fa[fm] = lds_read_b128(a_rd[s] + fm * 16 * (BK * 2));
#pragma unroll
            for (int fm = 0; fm < 4; fm++)
#pragma unroll
                for (int fn = 0; fn < 4; fn++)
                    acc[fm][fn] = __builtin_amdgcn_mfma_f32_16x16x32_f16(fb[fn], fa[fm], acc[fm][fn], 0, 0, 0);
        }
    }

    // ---- split k: this part's sums are added to C (only the launcher's f32 instantiation) ----
    // One atomic instruction per row of the wavefront's 64 x 64 block, 64 consecutive floats
    // (measured 190 G additions/s; in the accumulators' own layout -- 16 rows x 4 floats per
    // instruction -- 70 G/s): the block goes through a wavefront-private 17 KB of the LDS, which
    // is free once every wavefront is through its last k step.
    if constexpr (SPLIT) {
        constexpr uint32_t T_PITCH = 64 * 4 + 16;                 // bytes per row: rows 8 apart share banks, two at a time
        const uint32_t tbuf = smem_base + (uint32_t)wave * (64u * T_PITCH);
        __syncthreads();
#pragma unroll
        for (int fm = 0; fm < 4; fm++)
#pragma unroll
            for (int fn = 0; fn < 4; fn++)
                *(__attribute__((address_space(3))) floatx4*)(uintptr_t)(tbuf + (uint32_t)(fm * 16 + c_lrow) * T_PITCH + (uint32_t)(fn * 16 + c_lcol) * 4) = acc[fm][fn];
        const int rows_in = p.M - c_row0 < 64 ? p.M - c_row0 : 64;             // rows of the block inside C (may be <= 0)
        const bool col_in = c_col0 + lane < p.N;
        float* const cbase = reinterpret_cast<float*>(Cbase) + (int64_t)c_row0 * p.ldc + c_col0 + lane;
        for (int r = 0; r < rows_in; r++) {
            const float v = *(__attribute__((address_space(3))) const float*)(uintptr_t)(tbuf + (uint32_t)r * T_PITCH + 4u * lane);
            // a part that sums to zero leaves C alone (the memory's adders need not keep a subnormal C + 0)
            if (col_in && v != 0.0f) unsafeAtomicAdd(cbase + (int64_t)r * p.ldc, v);
        }
    } else {
        // ---- + C, + bias, ReLU, -> C: the wavefront's block goes through its part of the LDS ------
        constexpr uint32_t T_PITCH = 64 * 4 + 16;
        const uint32_t tbuf = smem_base + (uint32_t)wave * (64u * T_PITCH);
        __syncthreads();
#pragma unroll
        for (int fm = 0; fm < 4; fm++)
#pragma unroll
            for (int fn = 0; fn < 4; fn++)
                *(__attribute__((address_space(3))) floatx4*)(uintptr_t)(tbuf + (uint32_t)(fm * 16 + c_lrow) * T_PITCH + (uint32_t)(fn * 16 + c_lcol) * 4) = acc[fm][fn];
        asm volatile("" ::: "memory");                                // (a wavefront's LDS operations are carried out in order)
        float bias_v[VEC];
#pragma unroll
        for (int e = 0; e < VEC; e++) bias_v[e] = (p.bias && r_col_in) ? (float)reinterpret_cast<const CT*>(p.bias)[c_col0 + r_x + e] : 0.0f;
#pragma unroll
        for (int ps = 0; ps < PASSES; ps++) {
            ctv o;
#pragma unroll
            for (int v = 0; v < VEC; v += 4) {
                const floatx4 s4 = *(__attribute__((address_space(3))) const floatx4*)(uintptr_t)(tbuf + (uint32_t)(RPP * ps + r_row) * T_PITCH + (uint32_t)(r_x + v) * 4);
#pragma unroll
                for (int e = 0; e < 4; e++) o[v + e] = (CT)epilogue_value(s4[e] + (float)rin[ps][v + e], bias_v[v + e], p.relu);   // f16: one rounding, to nearest even
            }
            if (r_ok(ps)) *r_at(ps) = o;
        }
    }
}

int64_t grid_w4a128(int64_t M, int64_t N)
{
    const int64_t tm = (M + SBM - 1) / SBM, tn = (N + SBN - 1) / SBN;
    if (tm > 0 && tn > INT32_MAX / tm) return -1;
    return tm * tn;
}

// Split k, which XCD takes what (workgroup ids are dealt to the XCDs in turn).  Apart: the tiles of part 0, then those of part 1 and so on, in one
// order of which each XCD takes a contiguous slice, so that its workgroups share one or two parts' rows of B and k columns of A (with 16 parts, two a slice): a part's operands
// pass through fewer of the L2s ((256,4096,16384): 205 -> 153 MB from beyond them).  Otherwise part p of the t-th tile is workgroup p * tiles + t, each part's tiles dealt
// to the XCDs in slices: all parts of a tile on one XCD where the number of tiles is a multiple of 8 (the tile's column of B is then a narrow strip of every k row, and the XCD
// reads all of A), else shifted by the number of tiles from part to part.  Measured on 110 random problems, three sets of operands | from
// memory, the second order -> apart, us: (1024,1024,8192) 40.7 -> 29.7 | 40.9 -> 33.4, (300,1000,9000) 22.2 -> 19.6 | 24.9 -> 23.2, (512,512,8192)
// 16.6 -> 15.0 | 18.8 -> 18.4, (64,4096,4096) 14.6 -> 13.4 | 17.3 -> 17.2, (5,4096,8192) 15.2 -> 13.5 | 14.8 -> 13.6; equal where the
// parts are few.  Not with 17 to 255 rows where the operands together take more than 68 MB and have to come
// from memory: (64,8192,8192) 37.2 -> 40.3, (25,3800,12672) 22.8 -> 23.8, (216,8192,4096) 31.7 -> 32.1 | 30.5 -> 32.0 (30 tiles and 64 tiles alike; why was not looked for).
// The line is drawn wide: 128 and 192 rows at 8192^2 gain 1 to 2 % from memory (41.1 -> 40.6, 51.1 -> 50.0).  With up to 16 rows, or from two full tiles of
// rows on, it gains or is even: (1,8192,8192) 29.1 -> 27.0 and 28.1 -> 26.9, (8,13064,7104) 35.9 -> 37.2 in one session and 36.7 -> 36.2 in another, (256,4096,16384) 56.2 -> 54.7; 200
// random problems there 0.93 to 1.03 of the time from memory, in turn 0.83 to 1.04 but for four of 33 at 257 to 384 rows and 70 to 80 MB, where three sets just fill the
// last-level cache ((290,2568,14496) 41.9 -> 45.3 | 48.4 -> 47.4, (270,2520,15368) 11 % the other way round).
int parts_apart(const GemmArgs& a)
{
    const double mb = 2e-6 * (double)a.K * (double)(a.M + a.N);
    return mb <= 68.5 || a.M <= 16 || a.M >= 256;
}

int launch_w4a128(const GemmArgs& a)
{
    const int64_t g = grid_w4a128(a.M, a.N);
    if (g < 0) return GEMM_F16_ERR_SIZE;
    TiledParams p = make_tiled_params(a, SBM, SBN, 8);   // an XCD's 64 concurrent tiles form an 8 x 8 block of C
    // the parts of a split k loop add to C atomically: f32 C and no bias or activation, which would have to wait for the last part
    const int parts = (a.k_split > 1 && !a.c_is_f16 && !a.bias && !a.relu) ? a.k_split : 1;
    if (g * parts > INT32_MAX) return GEMM_F16_ERR_SIZE;
    p.k_split = parts;
    p.parts_apart = parts_apart(a);
    if (a.c_is_f16)
        hipLaunchKernelGGL((gemm_w4a128_kernel<half_t, false>), dim3((unsigned)g), dim3(256), 0, a.stream, p);
    else
    {
        if (parts > 1) hipLaunchKernelGGL((gemm_w4a128_kernel<float, true>), dim3((unsigned)(g * parts)), dim3(256), 0, a.stream, p);
        else           hipLaunchKernelGGL((gemm_w4a128_kernel<float, false>), dim3((unsigned)g), dim3(256), 0, a.stream, p);
    }
    return hipGetLastError() == hipSuccess ? GEMM_F16_OK : GEMM_F16_ERR_LAUNCH;
}

const GemmConfigDesc kW4a128 = {
    "w4a_128x128x64", SBM, SBN, BK, 4, 64, 64, W4A128_LDS, true, launch_w4a128, grid_w4a128};

}  // namespace

const GemmConfigDesc* deep_ring_config() { return &kW4a128; }
