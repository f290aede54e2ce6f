// Join count, R +=, many whole tiles of 256 x 256 and a long K: a persistent workgroup's tiles as ONE stream of stages.
//
// What bounded count_i8_dma_persistent_kernel here was the write-back of a tile (15 us beside 39 of matrix work, 10 of them waiting
// for R): no matrix instruction of the unit runs under it, because R is read then, the tile goes to R through the operands' ring,
// and the next tile's stages have to wait for the ring.  Here
//   * R is read during the K loop, four values per lane (K below 3392: eight) every three stages or more, and added to the
//     accumulators, so that the write-back is stores alone.  (More at once delay the stages' own loads, memory operations retire
//     in order: 8192^2 x 4096 208 us by eights, 204 by fours.  Three stages, so that a wait for operands finds them there.)
//   * a wave carries its 64 x 64 counts to R through 2 KB of LDS of its own, 16 rows of a block at a time: no barrier, and the ring
//     stays the stages'.  (Straight from the accumulators, 4 bytes per lane: 207 us against 206.  With the operands exchanged, so that a
//     lane has 16 bytes of a row: 315 to 460, rows in pieces of 32 bytes.)
//   * so the next tile's first three stages are requested by this one's last three, like any others; the two stages
//     after the stores wait past them, the third for them.
// All workgroups run in step: with half of the XCDs half a tile behind (the first tile in two passes, R read in both) 224 us.
//
// us, count_i8_dma_persistent_kernel / here: 8192^2 x 4096 218 / 205, x 3392 197 / 182, x 2048 156 / 147, 7168 x 8192 x 4096 210 / 196,
// 9216 x 8192 x 4096 258 / 247, 16384^2 x 4096 841 / 806 (three sets of matrices in turn 947 / 861), 16384 x 8192 x 4096 406 / 411 (488 / 433).
// Bound: 160 us of K loop (its matrix instructions alone are 131, its stream alone 123) and R, 537 MB read and written, beside the operands' 403 MB
// from beyond the L2s: 4.6 TB/s, where a large copy reaches 4.8.  By counters data return is busy for 88 % of the launch, the matrix cores
// for 53, LDS for 29; written without being read, 184 us.
//
// The tile, the layout of a stage in LDS, the fragments' reads and the place of the barrier are count_i8_dma.hip's.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "amulet_internal.h"

// the LDS-DMA asm below sets M0 itself and says so in its clobber list
#pragma clang diagnostic ignored "-Winline-asm"

namespace amulet {

typedef int v2i __attribute__((ext_vector_type(2)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef __attribute__((address_space(3))) v2i *lds_v2i_ptr;
typedef __attribute__((address_space(3))) void *lds_void_ptr;

constexpr int CS_TILE = 256, CS_BK = 64, CS_STAGES = 4, CS_WAVES = 16;
constexpr int CS_A_BYTES = CS_TILE * CS_BK, CS_STAGE_BYTES = 2 * CS_A_BYTES, CS_RING_BYTES = CS_STAGES * CS_STAGE_BYTES;
constexpr int CS_IMAGE_BYTES = 16 * 32 * 4;             // a wave's own: 16 rows of a 32 x 32 block
constexpr int CS_LDS_BYTES = CS_RING_BYTES + CS_WAVES * CS_IMAGE_BYTES;
constexpr int CS_LOADS = 2;                             // per wave and stage
constexpr int CS_STORES = 16;                           // per wave and tile
// Stages of a tile: two behind the last one's stores, three to a group of R's values, three ahead of the next tile's first
constexpr int cs_least_stages(int group) { return 2 + 3 * (64 / group) + 3; }
static_assert(cs_least_stages(8) * CS_BK == COUNT_STREAM_LEAST_K, "");

extern __shared__ __attribute__((aligned(16))) int8_t cs_smem[];

// GROUP: values of R that a lane reads at a time.  NT: R is written around the caches; it is read so always.
template <int GROUP, bool NT>
__global__ void __launch_bounds__(64 * CS_WAVES) __attribute__((amdgpu_waves_per_eu(4, 4)))
count_i8_stream_kernel(const CountArgs args)
{
    constexpr int GROUPS = 64 / GROUP;
    const int lane = (int)threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int wr = wave >> 2, wc = wave & 3, li = lane & 31, lh = lane >> 5;

    // the tiles of this workgroup: places slot, slot + n_slots, ... of its XCD's part of the tile order
    const int tiles_m = args.M / CS_TILE, tiles_n = args.N / CS_TILE;
    const int xcd = (int)blockIdx.x & 7, n_slots = (int)gridDim.x >> 3;
    const int places = (int)xcd_places(tiles_m, tiles_n);
    int place = (int)blockIdx.x >> 3;
    auto tile = [&](int &row0, int &col0) -> int {     // the first that exists from `place` on
        for (; place < places; place += n_slots) {
            int tm, tn;
            if (!xcd_tile(place * 8 + xcd, tiles_m, tiles_n, tm, tn)) continue;
            row0 = tm * CS_TILE;
            col0 = tn * CS_TILE;
            place += n_slots;
            return 1;
        }
        return 0;
    };

    // A stage's 32 KB: wave w brings rows 16 w .. of A and k-rows 4 w .. of B, 16 bytes per lane, to where the fragments' reads
    // find them without bank conflicts (the layout of count_i8_dma.hip).
    const int a_row = wave * 16 + (lane >> 2), b_row = wave * 4 + (lane >> 4);
    const uint32_t a_voff = (uint32_t)a_row * (uint32_t)args.lda + (uint32_t)((((lane & 3) ^ ((a_row >> 2) & 3))) * 16);
    const uint32_t b_voff = (uint32_t)b_row * (uint32_t)args.ldb + (uint32_t)(((lane & 15) ^ ((b_row & 7) << 1)) * 16);
    const uint32_t lds_wave = (uint32_t)(uintptr_t)(lds_void_ptr)cs_smem + (uint32_t)wave * 1024u;
    const int8_t *pa, *pb;                              // the next stage to request
    const int64_t b_step = (int64_t)CS_BK * args.ldb;
    // (`go` is 0 behind the last tile's stages; the branch is inside the asm: the stages stay one basic block)
    auto request = [&](int slot, int go) {
        const uint32_t dst = __builtin_amdgcn_readfirstlane(lds_wave + (uint32_t)(slot * CS_STAGE_BYTES));
        asm volatile("s_cmp_eq_u32 %[g], 0\n\ts_cbranch_scc1 1f\n\t"
                     "s_mov_b32 m0, %[d]\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %[av], %[a]\n\t"
                     "s_add_u32 m0, %[d], %[o]\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %[bv], %[b]\n1:"
                     :: [g] "s"(go), [d] "s"(dst), [o] "n"(CS_A_BYTES), [av] "v"(a_voff), [bv] "v"(b_voff), [a] "s"(pa), [b] "s"(pb)
                     : "memory", "m0", "scc");
        pa += CS_BK;
        pb += b_step;
    };

    // ---- fragments -------------------------------------------------------------------------
    const int arow = wr * 64 + li, tb = lane >> 4, ts = lane & 15, krow = 16 * (tb >> 1) + (ts >> 1);
    int a_off[2], b_off[2];
#pragma unroll
    for (int x = 0; x < 2; ++x) {
        a_off[x] = arow * CS_BK + ((2 * x + lh) ^ ((arow >> 2) & 3)) * 16;
        const int col = (wc * 2 + x) * 32 + 16 * (tb & 1) + 8 * (ts & 1);
        b_off[x] = CS_A_BYTES + krow * CS_TILE + ((col >> 4) ^ ((krow & 7) << 1)) * 16 + (col & 15);
    }
    auto read_frags = [&](int slot, int ks, v4i (&a)[2], v4i (&b)[2]) {
        const int8_t *st = cs_smem + slot * CS_STAGE_BYTES;
#pragma unroll
        for (int x = 0; x < 2; ++x) a[x] = *(const v4i *)(st + a_off[ks] + x * 2048);
#pragma unroll
        for (int x = 0; x < 2; ++x) {
            const int8_t *p = st + b_off[x] + ks * 8192;
            const v2i lo = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i_ptr)p);
            const v2i hi = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i_ptr)(p + 2048));
            b[x] = v4i{lo.x, lo.y, hi.x, hi.y};
        }
    };
    v16i acc[2][2];
    auto mma = [&](const v4i (&a)[2], const v4i (&b)[2]) {
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int y = 0; y < 2; ++y) acc[x][y] = __builtin_amdgcn_mfma_i32_32x32x32_i8(a[x], b[y], acc[x][y], 0, 0, 0);
    };

    v4i fa0[2], fb0[2], fa1[2], fb1[2];
    int slot = 0;
    // Stage s of the stream, whose first fragments are there: the wait for stage s + 1 and the barrier stand between its two halves
    // (count_i8_dma.hip).  WAIT: operations that may be under way behind stage s + 1's loads, if `open`, else none.  Stage s + 3 is
    // requested, into the slot that stage s - 1 has left, if `go`.  `landed` runs behind the wait, `more` behind the request.
    auto stage = [&](auto wait, int open, int go, auto landed, auto more) {
        const int next = (slot + 1) & (CS_STAGES - 1);
        read_frags(slot, 1, fa1, fb1);
        mma(fa0, fb0);
        __builtin_amdgcn_sched_barrier(0);
        if (__builtin_constant_p(open) && open)
            asm volatile("s_waitcnt vmcnt(%0)" ::"n"(decltype(wait)::value) : "memory");
        else
            asm volatile("s_cmp_eq_u32 %1, 0\n\ts_cbranch_scc0 1f\n\ts_waitcnt vmcnt(%2)\n1:\ts_waitcnt vmcnt(%0)"
                         ::"n"(decltype(wait)::value), "s"(open), "n"(decltype(wait)::value > CS_LOADS ? CS_LOADS : 0) : "memory", "scc");
        landed();
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        request((slot + 3) & (CS_STAGES - 1), go);
        more();
        read_frags(next, 0, fa0, fb0);
        __builtin_amdgcn_sched_barrier(0);
        mma(fa1, fb1);
        slot = next;
    };
    const auto nothing = []() {};
    const std::integral_constant<int, CS_LOADS> steady;
    const std::integral_constant<int, CS_LOADS + CS_STORES> behind_stores;
    const std::integral_constant<int, CS_LOADS + GROUP> behind_r;

    int row0, col0;
    if (!tile(row0, col0)) return;
    pa = args.A + (int64_t)row0 * args.lda;
    pb = args.B + col0;
#pragma unroll
    for (int d = 0; d < CS_STAGES - 1; ++d) request(d, 1);
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * CS_LOADS) : "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    read_frags(0, 0, fa0, fb0);

    const int n = args.K / CS_BK;
    int stored = 0;                                     // the last tile's stores are among the operations under way
    for (;;) {
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int y = 0; y < 2; ++y)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[x][y][v] = 0;
        // Two stages whose successors were requested ahead of the last tile's stores.
        stage(behind_stores, stored, 1, nothing, nothing);
        stage(behind_stores, stored, 1, nothing, nothing);
        int s = 2;
        const int last = n - 3;
        int rv[GROUP];
        auto add_r = [&](int q) {
#pragma unroll
            for (int j = 0; j < GROUP; ++j) {
                asm volatile("" : "+v"(rv[j]));
                const int e = q * GROUP + j;
                v16i &block = acc[e >> 5][(e >> 4) & 1];
                block[e & 15] = (int)((uint32_t)block[e & 15] + (uint32_t)rv[j]);
            }
        };
        // The loads are asm like the operands', awaited by the stages' own counts: three stages on, R's values stand ahead of what may
        // still be under way.  Nothing may touch their registers in between, which the language does not promise: tests/test_stream_registers.py
        // walks the assembly for it.  (121 vector registers by fours, 125 by eights, of 128; 35 and 27 scalars stand in lanes of one, none of
        // them in the loop of stages without loads of R.)
        const uint32_t r_voff = (uint32_t)(4 * lh) * (uint32_t)args.ldr * 4u + (uint32_t)li * 4u;
        const int32_t *r_rows = args.R + (int64_t)(row0 + wr * 64) * args.ldr + col0 + wc * 64;
        const int span = last - s;
#pragma unroll
        for (int q = 0; q < GROUPS; ++q) {
            const int end = 2 + span * (q + 1) / GROUPS;
            stage(steady, 1, 1, [&]() { if (q > 0) add_r(q - 1); },
                  [&]() {
#pragma unroll
                      for (int j = 0; j < GROUP; ++j) {
                          asm volatile("global_load_dword %0, %1, %2 nt" : "=v"(rv[j]) : "v"(r_voff), "s"(r_rows) : "memory");
                          // the accumulators' order: rows 0 .. 3, 8 .. 11, ... of a block, then the block beside or below
                          const int e = q * GROUP + j;
                          r_rows += (e & 3) < 3 ? args.ldr : (e & 15) < 15 ? 5 * args.ldr : (e & 16) == 0 ? 32 - 27 * args.ldr : 5 * args.ldr - 32;
                      }
                  });
            // (opaque, so that the addresses of all groups are not held at once)
            asm volatile("" : "+s"(r_rows));
            stage(behind_r, 1, 1, nothing, nothing);
            stage(behind_r, 1, 1, nothing, nothing);
            for (s += 3; s < end; ++s) stage(steady, 1, 1, nothing, nothing);
        }
        int next_row0 = 0, next_col0 = 0;
        const int more = tile(next_row0, next_col0);
        pa = args.A + (int64_t)next_row0 * args.lda;
        pb = args.B + next_col0;
#pragma unroll
        for (int d = 0; d < 3; ++d) stage(steady, more, more, nothing, nothing);
        add_r(GROUPS - 1);

        // ---- write-back ------------------------------------------------------------------------
        // (the lane made opaque: nothing of this is held during the stages)
        int l = lane;
        asm volatile("" : "+v"(l));
        int32_t *const img = (int32_t *)(cs_smem + CS_RING_BYTES + wave * CS_IMAGE_BYTES);
        const int w_at = (l >> 5) * 128 + (l & 31), swap = (l >> 5) * 32;
        const int r_at = ((l >> 3) ^ (l >> 5)) * 32 + (l & 7) * 4;
        const uint32_t r_off = ((uint32_t)(l >> 3) * (uint32_t)args.ldr + (uint32_t)(l & 7) * 4u) * 4u;
        char *const r_wave = (char *)(args.R + (int64_t)(row0 + wr * 64) * args.ldr + col0 + wc * 64);
#pragma unroll
        for (int x = 0; x < 2; ++x)
#pragma unroll
            for (int y = 0; y < 2; ++y)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
#pragma unroll
                    for (int v = 0; v < 8; ++v) {
                        const int r = 8 * (v >> 2) + (v & 3);       // + 4 in the upper half of the lanes
                        img[(w_at + r * 32) ^ swap] = acc[x][y][8 * h + v];
                    }
                    __builtin_amdgcn_wave_barrier();
                    asm volatile("" ::: "memory");
#pragma unroll
                    for (int i = 0; i < 2; ++i) {
                        const v4i c = *(const v4i *)(img + r_at + i * 256);
                        v4i *const at = (v4i *)(r_wave + ((int64_t)(x * 32 + h * 16 + i * 8) * args.ldr + y * 32) * 4 + r_off);
                        if (NT) __builtin_nontemporal_store(c, at);
                        else *at = c;
                    }
                    __builtin_amdgcn_wave_barrier();
                    asm volatile("" ::: "memory");
                }
        if (!more) return;
        row0 = next_row0;
        col0 = next_col0;
        stored = 1;
    }
}

// (a place for every workgroup; whole aligned tiles whose byte offsets fit 31 bits, as for the other streamed kernels, R's too)
bool count_i8_stream_eligible(const CountArgs &a)
{
    return !a.assign && !a.pers_named && compute_units() >= 8 && xcd_places(a.M / CS_TILE, a.N / CS_TILE) >= compute_units() / 8 && count_i8_dma_eligible(a, 4) && a.K / CS_BK >= cs_least_stages(8) && a.ldr <= 0x7fffffffLL / (4 * 64);
}

// Rows of R 16, 32 or 64 KB apart lie in the same channels of the memory system, and here all workgroups write theirs at the same time.
// Where there are many rows and K is short, count_i8_dma_persistent_kernel, whose phases spread the writes over time, is ahead: us, there / here,
// 16384 x 8192 x 2432 305 / 318 (rows 256 bytes longer 309 / 300), x 2560 317 / 340 (319 / 315), 24576 x 8192 x 2176 423 / 462 (430 / 436),
// 12288 x 8192 x 2560 245 / 256, 16384^2 x 2176 570 / 599 (615 / 598), 28672 x 4096 x 2560 300 / 328, 32768 x 4096 x 2432 323 / 358 (312 / 310).
// Not with fewer rows or a longer K -- 10240 x 8192 x 3072 227 / 222, 16384 x 8192 x 3392 365 / 366, x 4096 406 / 411 (three sets of matrices in turn
// 488 / 433), 16384^2 x 2560 654 / 644, 20480 x 4096 x 2560 1.03 times -- nor 128 KB apart: 12288 x 32768 x 2432 1002 / 961.
bool count_i8_stream_in_step_loses(const CountArgs &a)
{
    const int64_t pitch = 4 * a.ldr, tiles_m = a.Mwhole / CS_TILE, tiles = tiles_m * (a.N / CS_TILE);
    if ((pitch != 16384 && pitch != 32768 && pitch != 65536) || tiles < 832 || tiles % 8 != 0 || a.K < 2048) return false;
    return tiles_m >= (pitch == 16384 ? 96 : pitch == 32768 ? 48 : 40) && a.K < (pitch == 65536 ? 2560 : 3392);
}

template <int GROUP, bool NT>
static hipError_t launch_stream(const CountArgs &a, hipStream_t s, CountRan &ran)
{
    const int grid = compute_units() / 8 * 8;
    ran.workgroups = grid;
    ran.r_group = GROUP;
    ran.r_bypass = NT ? 1 : 0;
    static hipError_t granted = hipFuncSetAttribute(reinterpret_cast<const void *>(&count_i8_stream_kernel<GROUP, NT>), hipFuncAttributeMaxDynamicSharedMemorySize, CS_LDS_BYTES);
    if (granted != hipSuccess) return granted;
    if (forced_launch_failure()) return hipErrorLaunchFailure;
    hipLaunchKernelGGL((count_i8_stream_kernel<GROUP, NT>), dim3((unsigned)grid), dim3(64 * CS_WAVES), CS_LDS_BYTES, s, a);
    return hipGetLastError();
}

hipError_t launch_count_i8_stream(const CountArgs &a, hipStream_t s, CountRan &ran)
{
    // R written around the caches, so that it does not displace operands -- an R that a call finds there is worth less than the operands of
    // the calls around it -- except where a call's matrices fit the last-level cache (256 MiB) and there is little K to a tile, or where its
    // last round has few tiles and the tile kernels' smaller ones fill it better: there a call repeated on its matrices was slower than
    // with those kernels.  (Read around them always: 0.99 to 1.01 repeated, up to 1.25 with other matrices.)  us, kernels before / R written through
    // / around; on three sets of matrices in turn: 4352 x 4096 x 3392 83 / 78 / 86; 104 / 85 / 86, 5120 x 4096 x 2560 72 / 70 / 75; 88 / 78 / 75,
    // 8448 x 4096 x 4096 146 / 136 / 146; 188 / 168 / 149, 4608 x 4608 x 3072 77 / 74 / 80; 98 / 85 / 80, 16384 x 3328 x 1984 131 / 119 / 132;
    // 183 / 149 / 133; elsewhere around: 6144 x 8192 x 4096 170 / 145 / 156; 200 / 175 / 159, 7168 x 8192 x 2432 161 / 137 / 148; 161 / 167 / 150.
    // (Over 200 whole problems of 256 to 1100 tiles, against the kernels before: repeated 0.97 to 1.5 times as fast, 4 of them below 0.985; with other
    // matrices 1.0 to 1.5.)
    const int64_t units = compute_units(), tiles = (a.Mwhole / CS_TILE) * (a.N / CS_TILE), last = tiles % units;
    const double bytes = 4.0 * (double)a.Mwhole * (double)a.N + (double)a.K * ((double)a.Mwhole + (double)a.N);
    const bool around = bytes > 265e6 || (a.K >= 2560 && (tiles >= 832 || last == 0 || last > units / 2 || a.K >= (last > units / 4 ? 3392 : 4608)));
    if (a.K / CS_BK >= cs_least_stages(4)) return around ? launch_stream<4, true>(a, s, ran) : launch_stream<4, false>(a, s, ran);
    return around ? launch_stream<8, true>(a, s, ran) : launch_stream<8, false>(a, s, ran);
}

}  // namespace amulet
