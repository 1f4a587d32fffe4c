// Device-side helpers shared by the tuned kernels (gemm_tiled.hip,
// gemm_pingpong.hip): the direct global -> LDS copy, the two LDS fragment
// reads, the XCD-aware workgroup -> tile map.  gfx950 only.
#pragma once
#include "gemm_common.h"

namespace gemm_dev {

constexpr int BK = 64;             // k extent per LDS stage (f16 elements)

struct TiledParams {
    int M, N, K;
    const half_t* A; int64_t lda;
    const half_t* B; int64_t ldb;
    void* C; int64_t ldc;
    int tiles_m, tiles_n, group_m;
    int num_xcd;           // XCDs the workgroup ids are dealt to in turn (1: tiles in plain order)
    const void* bias;      // fused epilogue: N elements of C's type or nullptr; relu 0 / 1
    int relu;
    int stagger_ticks;     // late start: workgroups on odd XCDs start this many wall-clock ticks late (0: all at once)
    int first_generation;  // late start: workgroups that begin with the launch (only these wait)
    int k_split;           // five-stage 128 x 128 kernel: > 1 = a workgroup takes one tile and one of this many parts of the k loop, and adds to C atomically
    int parts_apart;       // ... 1: the parts of a tile on different XCDs; 0: workgroup b takes tile b % tiles, part b / tiles
};

// A launch whose C is larger than what the 256 MB last-level cache can keep reads and writes it with the
// non-temporal hint: C would push A and B out of the cache and not be there at the next call itself.
// Below, C = A B + C into one C again and again finds C in the cache, and the hint takes it
// away; the line lies where no use loses.  us without -> with, one C again | three sets of operands
// and C in turn: f32 (6142,4720,216) 116 MB 50 -> 69 | 68 -> 71, (6000,6000,1000) 144 MB 104 -> 120 | 127 -> 118,
// (16384,2304,768) 151 MB 79 -> 84 | 96 -> 83, (2656,20864,64) 222 MB 71 -> 88 | 99 -> 89, (8192,8192,1024)
// 268 MB 188 -> 172 | 194 -> 169 (but with a kernel that reads C after it 246 -> 253), (3087,32256,448) 398 MB
// 194 -> 175 | 198 -> 172; f16 (16384,3072,768) 101 MB 89 -> 92 | 99 -> 93, (5602,30592,384) 343 MB 223 -> 201 | 227 -> 200.
// (The hint on the loads alone or on the stores alone: up to 16 % slower on one C and 2 to 5 % faster on three.)
// Not below K = 256, where it costs more than it spares up to 340 MB ((4080,18944,64) f32 309 MB 119 -> 133 |
// 137 -> 134), not from K = 4096 on, where the traffic of C is a small part (8192^3 f32 795 -> 798), and
// not where rows of C begin within a 64-byte sector: (14910,2968,256) f32 at a pitch of 3032 91 -> 102.
constexpr double C_ONCE_BYTES = 300e6;
inline bool c_once(const GemmArgs& a)
{
    const int64_t size = a.c_is_f16 ? 2 : 4;
    return a.K >= 256 && a.K < 4096 && (double)a.M * (double)a.N * (double)size >= C_ONCE_BYTES && a.ldc * size % 64 == 0 && (uintptr_t)a.C % 64 == 0;
}

// The fields every launcher fills the same way: the problem, the tile grid for bm x bn tiles,
// and the tile order (group_m tile rows at a time; an XCD's 32 concurrent tiles should form a
// near-square block of C).
inline TiledParams make_tiled_params(const GemmArgs& a, int bm, int bn, int group_m)
{
    TiledParams p = {};
    p.M = (int)a.M; p.N = (int)a.N; p.K = (int)a.K;
    p.A = a.A; p.lda = a.lda; p.B = a.B; p.ldb = a.ldb; p.C = a.C; p.ldc = a.ldc;
    p.bias = a.bias; p.relu = a.relu;
    p.tiles_m = (int)((a.M + bm - 1) / bm);
    p.tiles_n = (int)((a.N + bn - 1) / bn);
    p.group_m = group_m < p.tiles_m ? group_m : p.tiles_m;
    p.num_xcd = chip().xcds;
    return p;
}

// The fused epilogue on one result: + bias, then ReLU written so that NaN and
// -0 pass through.
__device__ __forceinline__ float epilogue_value(float v, float bias, int relu)
{
    v += bias;
    return (relu && v < 0.0f) ? 0.0f : v;
}

typedef __attribute__((address_space(3))) void* lds_ptr_t;
typedef __attribute__((address_space(1))) const void* gbl_ptr_t;
typedef __attribute__((address_space(3))) shortx4* lds_s4_ptr_t;

// 16 bytes per lane, global -> LDS at lds_byte_addr (wave-uniform) + 16 * lane.
// The global address is base (wave-uniform, 64 bit) + byte_off (per lane, 32
// bit).  Written as inline assembly on purpose: the compiler cannot tell which
// LDS bytes an LDS-DMA load writes and would wait for ALL outstanding copies
// (vmcnt(0)) in front of every LDS read of the other buffer, serialising the
// prefetch with the MFMA phase.  The kernel orders these copies itself: an
// explicit vmcnt(0) and a barrier before a buffer is read.
__device__ __forceinline__ void async_copy16(const void* base, uint32_t byte_off, uint32_t lds_byte_addr)
{
    asm volatile("s_mov_b32 m0, %2\n\t"
                 "s_nop 0\n\t"
                 "global_load_lds_dwordx4 %0, %1"
                 :: "v"(byte_off), "s"(base), "s"(lds_byte_addr) : "memory", "m0");
}

// The same copy in two instructions that the caller separates by at least one other instruction
// (the wait state between a write of M0 and an LDS-DMA load): set_m0 puts base + imm into M0
// (imm must fold to a compile-time constant), async_copy16_m0 is the load.  Nothing in between
// may write M0; the kernels that use the pair issue nothing but MFMAs there.
__device__ __forceinline__ void set_m0(uint32_t base, uint32_t imm)
{
    asm volatile("s_add_u32 m0, %0, %1" :: "s"(base), "n"(imm) : "m0", "scc");
}
__device__ __forceinline__ void async_copy16_m0(const void* base, uint32_t byte_off)
{
    asm volatile("global_load_lds_dwordx4 %0, %1" :: "v"(byte_off), "s"(base) : "memory");
}

__device__ __forceinline__ half8 lds_read_b128(uint32_t addr)
{
    return *(__attribute__((address_space(3))) const half8*)(uintptr_t)addr;
}

__device__ __forceinline__ half4 lds_read_tr16(uint32_t addr)
{
    shortx4 v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4_ptr_t)(uintptr_t)addr);
    return __builtin_bit_cast(half4, v);
}

// The workgroup barrier between two phases of the phase-alternating kernels.
__device__ __forceinline__ void phase_barrier()
{
    // nothing may be scheduled across a phase boundary
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}

// Workgroup id -> position in an order of `num` items.  Ids are dealt to the XCDs
// round-robin; give XCD x the x-th contiguous slice of the order.
__device__ __forceinline__ int xcd_slice(int num, int num_xcd, int pid)
{
    const int q = num / num_xcd, r = num % num_xcd;
    const int x = pid % num_xcd;
    return x * q + (x < r ? x : r) + pid / num_xcd;
}

// The l-th tile of an order that walks group_m tile rows at a time, column by column.
__device__ __forceinline__ void tile_in_order(const TiledParams& p, int l, int& tile_m, int& tile_n)
{
    const int group_size = p.group_m * p.tiles_n;
    const int g = l / group_size;
    const int first_m = g * p.group_m;
    const int gm = (p.tiles_m - first_m < p.group_m) ? (p.tiles_m - first_m) : p.group_m;
    const int in_group = l % group_size;
    tile_m = first_m + in_group % gm;
    tile_n = in_group / gm;
}

// Workgroup id -> C tile.
__device__ __forceinline__ void tile_of_block(const TiledParams& p, int pid, int& tile_m, int& tile_n)
{
    tile_in_order(p, xcd_slice(p.tiles_m * p.tiles_n, p.num_xcd, pid), tile_m, tile_n);
}

// C tile <-> accumulators of one wavefront: FM x FN blocks of 32 x 32, block
// (fm, fn) at rows row0 + 32 fm, columns col0 + 32 fn (row0, col0 wave-uniform).
// Accumulator register i of lane l is row 8*(i/4) + 4*(l/32) + i%4, column l%32
// of its block.  Addresses are a wave-uniform row pointer plus one per-lane
// 32-bit offset, so that no per-element 64-bit address lives in registers.
// With `edge`, elements at rows >= M or columns >= N are read as 0 / not stored.
template <typename CT, int FM, int FN>
__device__ __forceinline__ void load_c_tile(floatx16 (&acc)[FM][FN], const CT* C, int64_t ldc,
                                            int row0, int col0, int lane, int M, int N, bool edge)
{
    const uint32_t voff = ((uint32_t)(4 * (lane >> 5)) * (uint32_t)ldc + (uint32_t)(lane & 31)) * (uint32_t)sizeof(CT);
    const int lrow = 4 * (lane >> 5), lcol = lane & 31;
#pragma unroll
    for (int fm = 0; fm < FM; fm++)
#pragma unroll
        for (int i = 0; i < 16; i++) {
            const int r = row0 + fm * 32 + 8 * (i / 4) + (i & 3);
            const char* rowp = reinterpret_cast<const char*>(C + (int64_t)r * ldc + col0);
#pragma unroll
            for (int fn = 0; fn < FN; fn++) {
                float v = 0.0f;
                if (!edge || (r + lrow < M && col0 + fn * 32 + lcol < N))
                    v = (float)*reinterpret_cast<const CT*>(rowp + voff + fn * 32 * sizeof(CT));
                acc[fm][fn][i] = v;
            }
        }
}

template <typename CT, int FM, int FN>
__device__ __forceinline__ void store_c_tile(const floatx16 (&acc)[FM][FN], CT* C, int64_t ldc,
                                             int row0, int col0, int lane, int M, int N, bool edge,
                                             const CT* bias, int relu)
{
    const uint32_t voff = ((uint32_t)(4 * (lane >> 5)) * (uint32_t)ldc + (uint32_t)(lane & 31)) * (uint32_t)sizeof(CT);
    const int lrow = 4 * (lane >> 5), lcol = lane & 31;
    float b[FN];
#pragma unroll
    for (int fn = 0; fn < FN; fn++) b[fn] = (bias && col0 + fn * 32 + lcol < N) ? (float)bias[col0 + fn * 32 + lcol] : 0.0f;
#pragma unroll
    for (int fm = 0; fm < FM; fm++)
#pragma unroll
        for (int i = 0; i < 16; i++) {
            const int r = row0 + fm * 32 + 8 * (i / 4) + (i & 3);
            char* rowp = reinterpret_cast<char*>(C + (int64_t)r * ldc + col0);
#pragma unroll
            for (int fn = 0; fn < FN; fn++)
                if (!edge || (r + lrow < M && col0 + fn * 32 + lcol < N))
                    *reinterpret_cast<CT*>(rowp + voff + fn * 32 * sizeof(CT)) = (CT)epilogue_value(acc[fm][fn][i], b[fn], relu);   // f16: one rounding, to nearest even
        }
}

// Accumulators formed with the operands exchanged (B fragment first) hold their block
// transposed: a lane owns 4 consecutive columns of one row of C per register group, so C moves
// 4 elements per lane and instruction (N is a multiple of 8 in the kernels that do this, so
// such a group lies entirely inside or outside C).  Vector accesses are only element-aligned.
template <typename CT> struct CVec4 {
    typedef CT type __attribute__((ext_vector_type(4), aligned(sizeof(CT))));
};

}  // namespace gemm_dev
