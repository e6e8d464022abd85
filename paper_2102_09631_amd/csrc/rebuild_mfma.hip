// Full gradient rebuild G = L^T R (Eq. 4) for bf16 factors on the gfx950 matrix cores.
//
// Both operands are stored with the contraction index K (the sample/token row)
// as the slow axis, while a bf16 MFMA operand wants each lane to hold eight
// consecutive K values of one output row/column.  Tiles are therefore staged in
// LDS exactly as they sit in memory ([k][column], 16-byte chunks XOR-swizzled by
// the row to spread banks) and read back with the LDS transpose-read, which
// hands every lane four K-consecutive values of its column.
//
// Two kernels: whole 256- or 128-tiles go straight from HBM into LDS (k_rebuild_bf16_dma, any K); every
// other shape is staged through registers with its edges clamped (k_rebuild_bf16).  Split-K partials
// are written as fp32 slabs and summed in fixed order by k_reduce_slabs, so results are reproducible
// bit for bit.
#include <type_traits>

#include "dad_internal.h"

namespace dad {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

namespace rb {
constexpr int TILE = 256;             // output tile edge
constexpr int BK = 32;                // K rows per pipeline stage
constexpr int ROWB = TILE * 2;        // bytes per LDS row
}  // namespace rb

// byte offset of 16-byte chunk `chunk` of row k inside an operand tile whose rows are ROWB bytes
template <int ROWB = rb::ROWB>
__device__ __forceinline__ int rb_lds_off(int k, int chunk) { return k * ROWB + ((chunk ^ ((k & 3) << 2)) << 4); }

typedef s16x4 __attribute__((address_space(3))) * lds_s16x4_ptr;

// Eight K-consecutive bf16 of column (m0 + lane%32), K rows kb + 8*(lane/32) .. +7, from a [k][col] tile.
template <int ROWB = rb::ROWB>
__device__ __forceinline__ bf16x8 rb_frag(const char* tile, int m0, int kb, int lane) {
    const int b = lane >> 4, s = lane & 15, j = s >> 2, g = s & 3;
    const int m = m0 + ((b & 1) << 4) + (g << 2);
    const int k = kb + ((b >> 1) << 3) + j;
    const char* p0 = tile + rb_lds_off<ROWB>(k, m >> 3) + ((g & 1) << 3);
    const char* p1 = tile + rb_lds_off<ROWB>(k + 4, m >> 3) + ((g & 1) << 3);
    s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(p0));
    s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(p1));
    s16x8 v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8, v);
}

// The XCD-aware order of the workgroups of a launch: hardware hands consecutive block ids to the eight
// XCDs round-robin; ids congruent mod 8 share an XCD and get consecutive logical ids, so that they walk
// neighbouring tiles of the same K chunk and hit each other's L2 lines.
__device__ __forceinline__ int rb_logical_id(int total) {
    const int per = total >> 3, main = per << 3;
    return (int)blockIdx.x < main ? (int)((blockIdx.x & 7) * per + (blockIdx.x >> 3)) : (int)blockIdx.x;
}

// ---------------------------------------------------------------------------------------------
// Any K, h_in, h_out (each operand at least eight elements).  128-tile, 2 x 2 waves of 64 x 64, 32 rows of K per stage.
// Tiles go global -> registers -> LDS with 16-byte loads at any element alignment (odd widths).
// What bounds it: the loads, about 30 bytes per clock and compute unit through the registers, and with two workgroups per unit
// the LDS.  So nothing else is left on the path: four stages of loads are in flight, fragments are read one contraction
// step ahead of their products (the last step of a stage behind the next one's barrier), and the loop over whole stages has no
// branch, as a wait behind one drains every load.  A stage of 32 rows takes 0.32 us where one workgroup has a unit to itself, 0.67
// for two; with one stage in flight and fragments read at the products it was 0.72.  13000 x 1000 x 1000: 300 us
// in one chunk, 132 so and 52 in eight; 3767 x 1300 x 2052: 92 -> 50 us.
// Columns beyond the matrix may hold anything, because their products land in results that are not
// stored: a chunk that crosses the end of a row simply reads on into the next one.  A chunk that
// would cross the end of the matrix is loaded from further down, and a stage that has such chunks or rows beyond K is mended in
// LDS before it is multiplied.
// Results leave with L as the matrix instruction's row operand: the 32 lanes of a half wave write 32
// consecutive columns of one row of G, whatever its alignment.
// ---------------------------------------------------------------------------------------------
typedef u32x4 u32x4_b2 __attribute__((aligned(2)));

namespace ra {
constexpr int TILE = 128, THREADS = 256, ROWB = TILE * 2;
constexpr int TILEB = rb::BK * ROWB, SLOTB = 2 * TILEB;  // an operand's tile, a stage
constexpr int SETS = 4;                                  // stages in flight in registers (two slots in LDS)
constexpr int LDS = 2 * SLOTB;
}  // namespace ra

// One workgroup's tile: `lid` is its logical index among the tiles_m * tiles_n * splits of this product.
__device__ __forceinline__ void rebuild_tile_any(const bf16_t* __restrict__ L, const bf16_t* __restrict__ R,
                                                 float* __restrict__ out, int64_t K, int h_in, int h_out,
                                                 int64_t chunk, int tiles_m, int tiles_n, int lid) {
    constexpr int TILE = ra::TILE, ROWB = ra::ROWB, BK = rb::BK, SETS = ra::SETS, TILEB = ra::TILEB, SLOTB = ra::SLOTB;
    constexpr int CPR = TILE / 8, RPP = ra::THREADS / CPR;  // chunks per row, rows per pass of the workgroup (two passes per tile)
    static_assert(2 * RPP == BK, "two loads per thread and operand cover a stage");
    // Rounds of four stages summed by the matrix instructions before they are added to the rest: one running sum over all of K
    // rounds at full height K / 16 times.  K = 3072, 1152 x 2101, error against fp64: 2.5e-7 with one sum,
    // 0.92e-7 folded every 256 rows.
    constexpr int FOLD = 2;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int tiles = tiles_m * tiles_n;
    const int split = lid / tiles, tile = lid - split * tiles;
    int pm, qn;
    if (tiles_m <= tiles_n) {
        pm = tile % tiles_m;
        qn = tile / tiles_m;
    } else {
        qn = tile % tiles_n;
        pm = tile / tiles_n;
    }
    const int p0 = pm * TILE, q0 = qn * TILE;
    const int64_t kbeg = (int64_t)split * chunk;
    const int64_t kend = (kbeg + chunk < K) ? kbeg + chunk : K;
    const int nk = (int)((kend - kbeg + BK - 1) / BK);

    const int c = t % CPR, r0 = t / CPR;  // this thread's chunk and first row of a tile
    const int pc = p0 + c * 8, qc = q0 + c * 8;
    const int64_t last_l = K * h_in - 8, last_r = K * h_out - 8;  // last element a 16-byte load may start at
    // Stages before `safe` lie inside the chunk and both matrices, the overrun of their last row's columns included.
    auto whole = [&](int h, int col0) {
        const int64_t room = K * h - (col0 + TILE), rows = room < 0 ? 0 : room / h + 1;  // rows k with k h + col0 + TILE <= K h
        return rows < kend ? rows : kend;
    };
    const int64_t safe_l = whole(h_in, p0), safe_r = whole(h_out, q0), safe_rows = (safe_l < safe_r ? safe_l : safe_r) - kbeg;
    const int safe = safe_rows <= 0 ? 0 : (int)(safe_rows / BK);

    u32x4 sl[SETS][2], sr[SETS][2];
    int ol[2], orr[2];  // offsets of the thread's loads in a stage
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        ol[i] = (r0 + RPP * i) * h_in + pc;
        orr[i] = (r0 + RPP * i) * h_out + qc;
    }
    // Loads of stage kt; one beyond the last repeats it, so that every wait is for a known number of younger loads.
    auto fetch = [&](int set, int kt) {
        const int64_t k0 = kbeg + (int64_t)(kt < nk ? kt : nk - 1) * BK;
        const int64_t bl = k0 * h_in, br = k0 * h_out;
        const int lim_l = last_l - bl < INT32_MAX ? (int)(last_l - bl) : INT32_MAX, lim_r = last_r - br < INT32_MAX ? (int)(last_r - br) : INT32_MAX;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            sl[set][i] = *reinterpret_cast<const u32x4_b2*>(L + bl + (ol[i] < lim_l ? ol[i] : lim_l));
            sr[set][i] = *reinterpret_cast<const u32x4_b2*>(R + br + (orr[i] < lim_r ? orr[i] : lim_r));
        }
    };
    auto put = [&](char* slot, int set, int i) {
        const int at = rb_lds_off<ROWB>(r0 + RPP * i, c);
        *reinterpret_cast<u32x4*>(slot + at) = sl[set][i];
        *reinterpret_cast<u32x4*>(slot + TILEB + at) = sr[set][i];
    };
    // Stage kt, landed in its slot and not whole: chunks that crossed the end of the matrix again element by element, rows beyond
    // the K chunk zeros.
    auto mend = [&](char* slot, int kt) {
#pragma unroll 1
        for (int i = 0; i < 4; ++i) {
            const bool left = i < 2;
            const bf16_t* const X = left ? L : R;
            const int h = left ? h_in : h_out, col = left ? pc : qc, row = r0 + RPP * (i & 1);
            const int64_t k = kbeg + (int64_t)kt * BK + row, at = k * h + col;
            if (k < kend && at <= (left ? last_l : last_r)) continue;
            uint32_t e[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) e[u] = k < kend && col + u < h ? X[at + u] : 0u;
            *reinterpret_cast<u32x4*>(slot + (left ? 0 : TILEB) + rb_lds_off<ROWB>(row, c)) =
                u32x4{e[0] | e[1] << 16, e[2] | e[3] << 16, e[4] | e[5] << 16, e[6] | e[7] << 16};
        }
    };

    f32x16 acc[2][2], sum[2][2];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[a][b][v] = sum[a][b][v] = 0.f;
    auto fold = [&]() {
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    sum[a][b][v] += acc[a][b][v];
                    acc[a][b][v] = 0.f;
                }
    };
    bf16x8 fa[2][2], fb[2][2];
#pragma unroll
    for (int a = 0; a < 2; ++a) fa[1][a] = fb[1][a] = bf16x8{0, 0, 0, 0, 0, 0, 0, 0};  // the step before the first multiplies zeros
    auto mma = [&](int set) {
#pragma unroll
        for (int a = 0; a < 2; ++a)
#pragma unroll
            for (int b = 0; b < 2; ++b) acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[set][a], fb[set][b], acc[a][b], 0, 0, 0);
    };
    auto step = [&](auto cur_c, int kt, bool inner) {  // inner: known to be whole
        constexpr int CUR = decltype(cur_c)::value, NEXT = (CUR + 1) % SETS;
        __syncthreads();  // stage kt is in LDS, and everyone is done with stage kt - 1
        char* const cur = smem + (CUR & 1) * SLOTB;
        char* const next = smem + (NEXT & 1) * SLOTB;
        if (!inner && kt >= safe) {
            mend(cur, kt);
            __syncthreads();
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
#pragma unroll
            for (int a = 0; a < 2; ++a) fa[ks][a] = rb_frag<ROWB>(cur, wm * 64 + a * 32, ks * 16, lane);
#pragma unroll
            for (int b = 0; b < 2; ++b) fb[ks][b] = rb_frag<ROWB>(cur + TILEB, wn * 64 + b * 32, ks * 16, lane);
            mma(ks ^ 1);
            put(next, NEXT, ks);
            if (ks == 1) fetch(NEXT, kt + 1 + SETS);
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);             // MFMA
                __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);             // LDS read
                if (m & 1) __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);  // LDS write
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    const std::integral_constant<int, 0> s0;
    const std::integral_constant<int, 1> s1;
    const std::integral_constant<int, 2> s2;
    const std::integral_constant<int, 3> s3;
#pragma unroll
    for (int i = 0; i < SETS; ++i) fetch(i, i);
    put(smem, 0, 0);
    put(smem, 0, 1);
    fetch(0, SETS);
    const int rounds = (safe < nk ? safe : nk) / SETS;
    int kt = 0;
    for (int done = 0; done < rounds;) {
        const int to = done + FOLD < rounds ? done + FOLD : rounds;
        for (; done < to; ++done, kt += SETS) {
            step(s0, kt, true);
            step(s1, kt + 1, true);
            step(s2, kt + 2, true);
            step(s3, kt + 3, true);
        }
        fold();
    }
    for (; kt < nk; kt += SETS) {
        step(s0, kt, false);
        if (kt + 1 < nk) step(s1, kt + 1, false);
        if (kt + 2 < nk) step(s2, kt + 2, false);
        if (kt + 3 < nk) step(s3, kt + 3, false);
        if (kt & SETS) fold();
    }
    mma(1);
    fold();

    // lane: column q = lane % 32, rows p = 8 (v / 4) + 4 (lane / 32) + v % 4 of each 32 x 32 block
    float* o = out + (int64_t)split * h_in * h_out;
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const int q = q0 + (wn * 2 + b) * 32 + (lane & 31);
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int p = p0 + (wm * 2 + a) * 32 + ((v >> 2) << 3) + ((lane >> 5) << 2) + (v & 3);
                if (p < h_in && q < h_out) o[(int64_t)p * h_out + q] = sum[a][b][v];
            }
        }
}

__global__ __launch_bounds__(ra::THREADS, 2) void k_rebuild_bf16(const bf16_t* __restrict__ L, const bf16_t* __restrict__ R,
                                                              float* __restrict__ out, int64_t K, int h_in, int h_out,
                                                              int64_t chunk, int tiles_m, int tiles_n, int total) {
    rebuild_tile_any(L, R, out, K, h_in, h_out, chunk, tiles_m, tiles_n, rb_logical_id(total));
}

// ---------------------------------------------------------------------------------------------
// Whole output tiles (any K): the operand tiles go from HBM straight into LDS (no register staging), through a ring of DMA_STAGES buffers, so three tiles per workgroup are
// in flight while the fourth is multiplied.  The XOR swizzle is applied on the global side: the
// lane that owns LDS chunk position c' of row k fetches global chunk c' ^ ((k & 3) << 2).
// The loads are issued through inline assembly because the compiler would otherwise wait for ALL
// outstanding LDS-bound loads before any LDS read; the waits are placed by hand instead.
//
// Eight waves (2 x 4, each 128 x 64 of the tile) rather than four: a wave can keep at most fifteen
// LDS reads in flight, and with one wave per SIMD the transpose-reads deliver only ~64 B/clk per CU,
// exactly what four 128 x 128 waves need at full MFMA rate; two waves per SIMD roughly double it.
namespace rb {
constexpr int DMA_STAGES = 4;
constexpr int DMA_LOADS = 4;  // 16-byte loads per thread per stage, for both tile sizes
}  // namespace rb

// T = tile edge, WM x WN waves, each (T/WM) x (T/WN) of the tile.  T = 256 with 2 x 4 waves is the
// kernel for large gradients.  T = 128 with 2 x 2 waves (two workgroups per CU) serves gradients with
// few 256-tiles, where filling the chip would otherwise take so many K chunks that their fp32
// partial slabs outweigh the operand reads.
// SRC is `const bf16_t*` (operands in one allocation each) or RowBlocks (the sites' blocks in
// place, the same row split for both operands, every block a multiple of 256 rows): a K chunk may
// span blocks, and the operand pointers jump at a block's end.
// TAIL: K is not a multiple of BK.  The rows of the last stage beyond K repeat row K - 1 and are zeroed in LDS before they are
// multiplied.  Whole K has an instance without that code: in the one loop of both it cost every product 4 to 7 %
// (65536 x 1024 x 4096: 484 -> 504 us, zero factors 350 -> 368 us; 242 -> 250 VGPRs, 32 -> 52 SGPRs).  Row blocks are whole
// stages, but their one instance has the zeroing (never entered): the compiler's schedule with it is the better one there
// (16 blocks of 16384 x 1280 x 5120: 2926 us with it, 2972 to 3008 without; smaller products equal).
// With 128-tiles such a K also adds every 256 rows to a second accumulator, as k_rebuild_bf16 does and for its reason
// (3077 x 1152 x 2176, error against fp64: 2.7e-7 with one running sum over a chunk, 0.97e-7 folded, fp32 FMA kernel before
// 1.4e-7; 20011 x 1152 x 2176: 121 -> 129 us, FMA kernel 1470 us); 256-tiles have no registers for it.
// One workgroup's tile: `lid` is its logical index among the tiles_m * tiles_n * splits of this product.
template <int T, int WM, int WN, typename SRC, bool TAIL>
__device__ __forceinline__ void rebuild_tile_dma(const SRC& L, const SRC& R, float* __restrict__ out, int64_t K, int h_in,
                                                 int h_out, int64_t chunk, int tiles_m, int tiles_n, int lid) {
    constexpr int WAVES = WM * WN;
    constexpr int FA = T / (32 * WM), FB = T / (32 * WN);  // 32-wide fragments per wave
    constexpr int ROWB = T * 2;                            // bytes per LDS row
    constexpr int TILEB = rb::BK * ROWB;
    constexpr int STAGEB = 2 * TILEB;
    constexpr int CPR = ROWB / 16;                         // 16-byte chunks per row
    constexpr int RPI = 64 / CPR;                          // tile rows covered by one load of a wave
    static_assert(rb::BK == 2 * RPI * WAVES, "two loads per wave and operand cover a stage");
    constexpr bool RAGGED = TAIL && std::is_pointer<SRC>::value;  // K may end inside a stage
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int wm = wave / WN, wn = wave % WN;

    const int tiles = tiles_m * tiles_n;
    const int split = lid / tiles, tile = lid - split * tiles;
    int pm, qn;
    if (tiles_m <= tiles_n) {
        pm = tile % tiles_m;
        qn = tile / tiles_m;
    } else {
        qn = tile % tiles_n;
        pm = tile / tiles_n;
    }
    const int p0 = pm * T, q0 = qn * T;
    const int64_t kbeg = (int64_t)split * chunk;
    const int64_t kend = (kbeg + chunk < K) ? kbeg + chunk : K;
    const int nk = (int)((kend - kbeg + (TAIL ? rb::BK - 1 : 0)) / rb::BK);
    const int tail = TAIL ? (int)((int64_t)nk * rb::BK - (kend - kbeg)) : 0;  // rows of the last stage beyond K

    // this lane's two rows per operand tile: row = 2*RPI*wave + RPI*i + lane/CPR, LDS chunk position lane%CPR
    RowCursor cur_l, cur_r;
    const char* l0 = row_address(L, kbeg, (int64_t)h_in * 2, cur_l);
    const char* r0 = row_address(R, kbeg, (int64_t)h_out * 2, cur_r);
    int64_t row_next = kbeg;  // first row of the next tile to be issued
    const char* gl[2];
    const char* gr[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int row = 2 * RPI * wave + RPI * i + lane / CPR;
        const int c = (lane % CPR) ^ ((row & 3) << 2);
        gl[i] = l0 + (row * (int64_t)h_in + p0 + c * 8) * 2;
        gr[i] = r0 + (row * (int64_t)h_out + q0 + c * 8) * 2;
    }
    const int64_t adv_l = (int64_t)rb::BK * h_in * 2, adv_r = (int64_t)rb::BK * h_out * 2;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem;

    auto issue = [&](int stage) {  // loads the next tile in sequence into ring slot `stage`
        // wave-uniform by construction; readfirstlane lets the compiler keep it in a scalar register
        const uint32_t base = __builtin_amdgcn_readfirstlane(lds0 + stage * STAGEB + (2 * RPI * wave) * ROWB);
        if constexpr (!std::is_pointer<SRC>::value) {
            if (row_next == cur_l.end) {
                const int64_t jl = block_jump(L, (int64_t)h_in * 2, cur_l);
                const int64_t jr = block_jump(R, (int64_t)h_out * 2, cur_r);
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    gl[i] += jl;
                    gr[i] += jr;
                }
            }
            row_next += rb::BK;
        }
        if constexpr (RAGGED) {
            if (row_next + rb::BK > kend) {
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const int64_t over = row_next + 2 * RPI * wave + RPI * i + lane / CPR - (kend - 1);
                    if (over > 0) {
                        gl[i] -= over * h_in * 2;
                        gr[i] -= over * h_out * 2;
                    }
                }
            }
            row_next += rb::BK;
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            dma16(gl[i], base + RPI * i * ROWB);
            gl[i] += adv_l;
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            dma16(gr[i], base + TILEB + RPI * i * ROWB);
            gr[i] += adv_r;
        }
    };

    f32x16 acc[FA][FB];
#pragma unroll
    for (int a = 0; a < FA; ++a)
#pragma unroll
        for (int b = 0; b < FB; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[a][b][v] = 0.f;

    constexpr bool FOLD = RAGGED && T == 128;
    f32x16 sum[FOLD ? FA : 1][FOLD ? FB : 1];
    auto fold = [&](bool first) {
        if constexpr (FOLD) {
#pragma unroll
            for (int a = 0; a < FA; ++a)
#pragma unroll
                for (int b = 0; b < FB; ++b)
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        sum[a][b][v] = first ? acc[a][b][v] : sum[a][b][v] + acc[a][b][v];
                        acc[a][b][v] = 0.f;
                    }
        }
    };
    fold(true);

#pragma unroll
    for (int s = 0; s < rb::DMA_STAGES - 1; ++s)
        if (s < nk) issue(s);

    // Each K tile is two MFMA K-steps (ks = 0, 1) with fragment sets 0 and 1.  The second step of a
    // tile is multiplied after the next tile's barrier, so the matrix cores have independent MFMAs to
    // chew on while the first fragments of the new tile travel from LDS:
    //   barrier | DMA(kt+3) | read set0(kt,0) x MFMA set1(kt-1,1) | read set1(kt,1) x MFMA set0(kt,0) | ...
    // where "x" is an instruction-by-instruction interleave: one or two fragment reads between
    // consecutive MFMAs (measured 6-7 % faster than reads and MFMAs in blocks: 67 % instead of 60 % of
    // peak on all-zero operands, 49 % instead of 46 % on the benchmark's).
    bf16x8 fa0[FA], fb0[FB], fa1[FA], fb1[FB];
    // set 1 starts as zeros, so that the first tile's "previous K-step" multiplies into zero accumulators
#pragma unroll
    for (int a = 0; a < FA; ++a) fa1[a] = bf16x8{0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int b = 0; b < FB; ++b) fb1[b] = bf16x8{0, 0, 0, 0, 0, 0, 0, 0};
    auto read_frags = [&](bf16x8 (&fa)[FA], bf16x8 (&fb)[FB], const char* tl, int ks) {
        const char* tr = tl + TILEB;
#pragma unroll
        for (int a = 0; a < FA; ++a) fa[a] = rb_frag<ROWB>(tl, wm * (FA * 32) + a * 32, ks * 16, lane);
#pragma unroll
        for (int b = 0; b < FB; ++b) fb[b] = rb_frag<ROWB>(tr, wn * (FB * 32) + b * 32, ks * 16, lane);
    };
    auto mma = [&](const bf16x8 (&fa)[FA], const bf16x8 (&fb)[FB]) {
#pragma unroll
        for (int a = 0; a < FA; ++a)
#pragma unroll
            for (int b = 0; b < FB; ++b)
                // R fragment as the MFMA's row operand: each lane then owns four consecutive q of one p
                acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[b], fa[a], acc[a][b], 0, 0, 0);
    };

    // One K tile; STAGE is a compile-time ring slot so every LDS address is lane offset + constant.
    auto step = [&](int kt, auto stage_c) {
        constexpr int STAGE = decltype(stage_c)::value;
        // tile kt has landed once at most DMA_STAGES-2 younger tiles are outstanding
        // everyone's part of tile kt is in LDS, and tile kt-1's slot is free
        if (kt + rb::DMA_STAGES - 2 < nk)
            tile_barrier<rb::DMA_LOADS * (rb::DMA_STAGES - 2)>();
        else
            tile_barrier<0>();
        if (kt + rb::DMA_STAGES - 1 < nk) issue((STAGE + rb::DMA_STAGES - 1) % rb::DMA_STAGES);
        const char* tl = smem + STAGE * STAGEB;
        if constexpr (TAIL) {
            if (tail && kt == nk - 1) {
                for (int e = t; e < tail * CPR; e += 64 * WAVES)
#pragma unroll
                    for (int op = 0; op < 2; ++op)
                        *reinterpret_cast<u32x4*>(smem + STAGE * STAGEB + op * TILEB + (rb::BK - tail) * ROWB + e * 16) = u32x4{0, 0, 0, 0};
                __syncthreads();
            }
        }
        constexpr int NR = 2 * (FA + FB), NM = FA * FB;  // LDS reads and MFMAs per K-step
        __builtin_amdgcn_sched_barrier(0);
        read_frags(fa0, fb0, tl, 0);
        mma(fa1, fb1);
        interleave_reads_mfma<NR, NM, true>();
        __builtin_amdgcn_sched_barrier(0);
        read_frags(fa1, fb1, tl, 1);
        mma(fa0, fb0);
        interleave_reads_mfma<NR, NM, false>();
        __builtin_amdgcn_sched_barrier(0);
    };
    for (int kt = 0; kt < nk; kt += rb::DMA_STAGES) {
        step(kt, std::integral_constant<int, 0>{});
        if (kt + 1 < nk) step(kt + 1, std::integral_constant<int, 1>{});
        if (kt + 2 < nk) step(kt + 2, std::integral_constant<int, 2>{});
        if (kt + 3 < nk) step(kt + 3, std::integral_constant<int, 3>{});
        if (FOLD && (kt & rb::DMA_STAGES)) fold(false);
    }
    if (nk > 0) mma(fa1, fb1);
    fold(false);

    // D[q][p] layout: lane holds p = lane % 32 and q = 8*g + 4*(lane/32) + 0..3 for g = 0..3: 16-byte stores
    float* o = out + (int64_t)split * h_in * h_out;
#pragma unroll
    for (int a = 0; a < FA; ++a)
#pragma unroll
        for (int b = 0; b < FB; ++b) {
            const int p = p0 + wm * (FA * 32) + a * 32 + (lane & 31);
            const int qb = q0 + wn * (FB * 32) + b * 32 + ((lane >> 5) << 2);
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const f32x16& x = FOLD ? sum[FOLD ? a : 0][FOLD ? b : 0] : acc[a][b];
                f32x4 v4 = {x[4 * g], x[4 * g + 1], x[4 * g + 2], x[4 * g + 3]};
                *reinterpret_cast<f32x4*>(o + (int64_t)p * h_out + qb + 8 * g) = v4;
            }
        }
}

template <int T, int WM, int WN, typename SRC, bool TAIL>
__global__ __launch_bounds__(64 * WM * WN) void k_rebuild_bf16_dma(const SRC L, const SRC R,
                                                                  float* __restrict__ out, int64_t K, int h_in,
                                                                  int h_out, int64_t chunk, int tiles_m,
                                                                  int tiles_n, int total) {
    rebuild_tile_dma<T, WM, WN, SRC, TAIL>(L, R, out, K, h_in, h_out, chunk, tiles_m, tiles_n, rb_logical_id(total));
}

// Several products in one launch (the full gradients of the layers of a block): gradients with few
// 256-tiles fill the chip together, so each needs fewer K chunks and writes fewer fp32 slabs.
namespace rb {
constexpr int MAX_JOBS = 16;
}
struct RebuildJob {
    const bf16_t* L;
    const bf16_t* R;
    float* out;  // G, or the first of its slabs
    int64_t K, chunk;
    int h_in, h_out, tiles_m, tiles_n;
    int total;  // workgroups
};
struct RebuildJobs {
    int first_block[rb::MAX_JOBS];  // first logical id of each job; entries beyond the last job hold INT_MAX
    RebuildJob j[rb::MAX_JOBS];
};

template <int T, int WM, int WN, bool TAIL>
__global__ __launch_bounds__(64 * WM * WN) void k_rebuild_bf16_dma_jobs(RebuildJobs tb, int total) {
    const int lid = rb_logical_id(total);
    int ji = 0;
#pragma unroll
    for (int i = 1; i < rb::MAX_JOBS; ++i) ji += tb.first_block[i] <= lid ? 1 : 0;
    const RebuildJob& jb = tb.j[ji];
    const bf16_t* L = jb.L;
    const bf16_t* R = jb.R;
    rebuild_tile_dma<T, WM, WN, const bf16_t*, TAIL>(L, R, jb.out, jb.K, jb.h_in, jb.h_out, jb.chunk, jb.tiles_m, jb.tiles_n,
                                                     lid - tb.first_block[ji]);
}


// Products with plans of their own (the M of several reductions): their workgroups differ in length, so every product is dealt to all
// eight XCDs in equal shares, the one with the longest workgroups first; an XCD's share of a product is a contiguous run of its logical
// ids.  first_block counts the workgroups of one XCD.
__device__ __forceinline__ int rb_own_id(const RebuildJobs& tb, int* job) {
    const int at = (int)(blockIdx.x >> 3);
    int ji = 0;
#pragma unroll
    for (int i = 1; i < rb::MAX_JOBS; ++i) ji += tb.first_block[i] <= at ? 1 : 0;
    *job = ji;
    const int total = tb.j[ji].total, lid = (int)(blockIdx.x & 7) * ((total + 7) >> 3) + at - tb.first_block[ji];
    return lid < total ? lid : -1;
}

template <int T, int WM, int WN, bool TAIL>
__global__ __launch_bounds__(64 * WM * WN) void k_rebuild_bf16_dma_own(RebuildJobs tb) {
    int ji;
    const int lid = rb_own_id(tb, &ji);
    if (lid < 0) return;
    const RebuildJob& jb = tb.j[ji];
    const bf16_t* L = jb.L;
    const bf16_t* R = jb.R;
    rebuild_tile_dma<T, WM, WN, const bf16_t*, TAIL>(L, R, jb.out, jb.K, jb.h_in, jb.h_out, jb.chunk, jb.tiles_m, jb.tiles_n, lid);
}

__global__ __launch_bounds__(ra::THREADS, 2) void k_rebuild_bf16_own(RebuildJobs tb) {
    int ji;
    const int lid = rb_own_id(tb, &ji);
    if (lid < 0) return;
    const RebuildJob& jb = tb.j[ji];
    rebuild_tile_any(jb.L, jb.R, jb.out, jb.K, jb.h_in, jb.h_out, jb.chunk, jb.tiles_m, jb.tiles_n, lid);
}



// The direct-to-LDS kernel takes whole output tiles.
static bool rebuild_whole_tiles(int64_t K, int64_t h_in, int64_t h_out) {
    return K >= 256 && h_in % 128 == 0 && h_out % 128 == 0 && h_in <= (1 << 20) && h_out <= (1 << 20);
}

// Every bf16 product but those of an operand shorter than one 16-byte load.
bool rebuild_fast_ok(int64_t K, int64_t h_in, int64_t h_out, dad_dtype dt) {
    return dt == DAD_BF16 && K * h_in >= 8 && K * h_out >= 8;
}

// Most K chunks of the register-staged kernel.  Every chunk is a slab of the workspace, and a workspace that was large enough for a
// product stays large enough: the limit is what paid at 3 us and 0.5 us per 64 rows of a round of two workgroups per unit, which is
// what the size query goes by.  36 shapes, without it and with it: mostly alike, 15224 x 3602 x 1237 245 and 263 us (four more slabs of
// 18 MB), 743 x 128 x 1269 13 and 16, 13131 x 4375 x 2343 507 and 435.
static int64_t rebuild_any_slabs(int64_t K, int64_t tiles, int64_t h_in, int64_t h_out) {
    double best_t = 0.0;
    int64_t best = 1;
    for (int64_t s = 1; s <= 64; ++s) {
        if (s > 1 && K / s < 4 * rb::BK) break;
        const double stages = (double)ceil_div(ceil_div(K, s), 2 * rb::BK);
        double t = (double)ceil_div(tiles * s, 2 * CU_COUNT) * (3.0 + 0.5 * stages);
        if (s > 1) t += 4.0 + (2.0 * s + 1.0) * h_in * h_out * 4.0 / 4e6;
        if (s == 1 || t < best_t * 0.98) best_t = t, best = s;
    }
    return ceil_div(K, (int64_t)align_up((size_t)ceil_div(K, best), 2 * rb::BK));
}

// K chunks of the register-staged kernel, by a time in us.  A stage takes 0.32 us and up to 0.1 more as the units fill, 0.67 for
// two workgroups of a unit; more than one chunk adds the slab traffic and the launch that sums it.
static SplitPlan rebuild_any_split(int64_t K, int64_t h_in, int64_t h_out, int limit) {
    const int64_t tiles = ceil_div(h_in, ra::TILE) * ceil_div(h_out, ra::TILE);
    int64_t most = rebuild_any_slabs(K, tiles, h_in, h_out);
    if (most > limit) most = limit;
    double best_t = 0.0;
    int64_t best = 1;
    for (int64_t s = 1; s <= most; ++s) {
        const double stages = (double)ceil_div(ceil_div(K, s), rb::BK), wg = (double)(tiles * s);
        const double stage = wg <= CU_COUNT ? 0.32 + 0.1 * wg / CU_COUNT : 0.67 * (double)ceil_div(tiles * s, 2 * CU_COUNT);
        double t = 6.0 + stages * stage;
        if (s > 1) t += 3.5 + (2.0 * s + 1.0) * h_in * h_out * 4.0 / 6e6;
        if (s == 1 || t < best_t * 0.98) best_t = t, best = s;
    }
    SplitPlan sp;
    sp.chunk = (int64_t)align_up((size_t)ceil_div(K, best), rb::BK);
    sp.splits = (int)ceil_div(K, sp.chunk);
    return sp;
}

// A stage of 32 rows for a workgroup of its kernel, by how many of them share a unit, as fitted to 400 products on the way to a
// reduction.
ProductTime rebuild_bf16_time(int64_t K, int64_t h_in, int64_t h_out, const RebuildPlan& p) {
    const int tile = p.tile ? p.tile : ra::TILE, s = p.split.splits;
    const int64_t wg = ceil_div(h_in, tile) * ceil_div(h_out, tile) * s, slots = tile == 256 ? CU_COUNT : 2 * CU_COUNT;
    // Of a whole round.  128-tiles of a larger product drift apart in K and lose each other's lines: 0.41 us at 100 MB of operands, 0.49 at 250,
    // 0.60 at 500, 0.72 at 800 (131072 x 1536 x 1536 in three chunks: 986 us).
    const double mb = (double)K * (h_in + h_out) * 2e-6;
    const double full = p.tile == 0 ? 0.48 : p.tile == 128 ? 0.41 + (mb > 100.0 ? 0.0005 * (mb - 100.0) : 0.0) : 0.89;
    const double first = p.tile == 0 ? 0.23 + 0.07 * wg / CU_COUNT : p.tile == 128 ? (p.fine ? 0.34 : 0.32) : full;  // one workgroup to a unit
    const double stages = (double)ceil_div(p.split.chunk, rb::BK), slabs = s == 1 ? 0.0 : 0.24 * (2.0 * s + 1.0) * h_in * h_out * 4e-6;
    return ProductTime{(p.tile == 0 ? 4.3 : 0.5) + slabs + (s == 1 ? 0.0 : 2.5) + stages * (wg <= CU_COUNT ? first : full * (double)ceil_div(wg, slots)),
                       slabs + stages * full * (double)wg / (double)slots};
}

// Score of a tiling: share of the CU slots that whole rounds of workgroups fill, discounted by the
// fp32 partial traffic (splits * h_in * h_out * 4 bytes written, read, and the result written) next
// to the operand reads, and for 128-tiles by their doubled L2->LDS traffic per flop.
static double rebuild_score(int64_t K, int64_t h_in, int64_t h_out, int tile, int s) {
    const int64_t wg = (h_in / tile) * (h_out / tile) * s;
    const int64_t slots = tile == 256 ? 256 : 512;
    const double eff = (double)wg / (double)(ceil_div(wg, slots) * slots);
    const double ops = (double)K * (h_in + h_out) * 2.0;
    const double extra = s > 1 ? (2.0 * s + 1.0) * h_in * h_out * 4.0 : 0.0;
    return eff / (1.0 + extra / ops) * (tile == 256 ? 1.0 : 0.8);
}

// Tile edge and number of K chunks, `most` at most; tile 0: the register-staged kernel.
SplitPlan rebuild_fast_split(int64_t K, int64_t h_in, int64_t h_out, int* tile_out, int most, bool fine) {
    if (!rebuild_whole_tiles(K, h_in, h_out)) {
        *tile_out = 0;
        return rebuild_any_split(K, h_in, h_out, most);
    }
    int best = 1, best_tile = 0;
    double best_score = -1.0;
    for (int tile : {256, 128}) {
        if (h_in % tile || h_out % tile || (fine && tile == 256)) continue;  // 256-tiles have no registers for a second sum
        for (int s = 1; s <= most; ++s) {
            if (s > 1 && K / s < 1024) break;
            const double score = rebuild_score(K, h_in, h_out, tile, s);
            if (score > best_score * 1.02) {
                best_score = score;
                best = s;
                best_tile = tile;
            }
        }
    }
    SplitPlan sp;
    sp.chunk = (int64_t)align_up((size_t)ceil_div(K, best), rb::BK);
    sp.splits = (int)ceil_div(K, sp.chunk);
    *tile_out = best_tile;
    return sp;
}

template <int T, int WM, int WN>
static dad_status launch_rebuild_dma(const void* L, const void* R, const RowBlocks* lb, const RowBlocks* rbk, float* dst,
                                     int64_t K, int64_t h_in, int64_t h_out, SplitPlan sp, bool fine, hipStream_t s) {
    const int lds = rb::DMA_STAGES * 2 * rb::BK * T * 2;
    const int tm = (int)(h_in / T), tn = (int)(h_out / T);
    const int total = tm * tn * sp.splits;
    ProfScope prof(KID_REBUILD_BF16_DMA, s);
    const dim3 grid((unsigned)total), block(64 * WM * WN);
    const bf16_t *l = static_cast<const bf16_t*>(L), *r = static_cast<const bf16_t*>(R);
    if (lb)
        hipLaunchKernelGGL((k_rebuild_bf16_dma<T, WM, WN, RowBlocks, true>), grid, block, lds, s, *lb, *rbk, dst, K, (int)h_in,
                           (int)h_out, sp.chunk, tm, tn, total);
    else if (K % rb::BK == 0 && !fine)
        hipLaunchKernelGGL((k_rebuild_bf16_dma<T, WM, WN, const bf16_t*, false>), grid, block, lds, s, l, r, dst, K, (int)h_in,
                           (int)h_out, sp.chunk, tm, tn, total);
    else
        hipLaunchKernelGGL((k_rebuild_bf16_dma<T, WM, WN, const bf16_t*, true>), grid, block, lds, s, l, r, dst, K, (int)h_in,
                           (int)h_out, sp.chunk, tm, tn, total);
    DAD_LAUNCH_CHECK();
    return DAD_OK;
}

// lb / rbk, when not null, give both operands as row blocks (L and R are then unused); only the
// direct-to-LDS kernel reads blocks.
dad_status fast_rebuild(const void* L, const void* R, const RowBlocks* lb, const RowBlocks* rbk, int64_t K, int64_t h_in,
                        int64_t h_out, float* G, float* partials, SplitPlan sp, int tile, hipStream_t s, bool fine) {
    float* dst = sp.splits == 1 ? G : partials;
    dad_status rc;
    if ((lb != nullptr) != (rbk != nullptr) || (lb && tile == 0)) return DAD_ERR_SHAPE;
    if (tile != 0) {
        rc = tile == 128 ? launch_rebuild_dma<128, 2, 2>(L, R, lb, rbk, dst, K, h_in, h_out, sp, fine, s)
                         : launch_rebuild_dma<256, 2, 4>(L, R, lb, rbk, dst, K, h_in, h_out, sp, fine, s);
        if (rc != DAD_OK) return rc;
    } else {
        const int tm = (int)ceil_div(h_in, ra::TILE), tn = (int)ceil_div(h_out, ra::TILE);
        const int total = tm * tn * sp.splits;
        ProfScope prof(KID_REBUILD_BF16, s);
        hipLaunchKernelGGL(k_rebuild_bf16, dim3((unsigned)total), dim3(ra::THREADS), ra::LDS, s,
                           (const bf16_t*)L, (const bf16_t*)R, dst, K, (int)h_in, (int)h_out, sp.chunk, tm, tn, total);
        DAD_LAUNCH_CHECK();
    }
    if (sp.splits > 1) return reduce_slabs(partials, G, h_in * h_out, sp.splits, s);
    return DAD_OK;
}

// True when a product can join a launch of several: whole 256-tiles.
bool rebuild_group_ok(int64_t K, int64_t h_in, int64_t h_out, dad_dtype dt) {
    return dt == DAD_BF16 && K >= 256 && h_in % 256 == 0 && h_out % 256 == 0 && h_in <= (1 << 20) &&
           h_out <= (1 << 20);
}

// Number of K chunks for n products launched together (the same for all of them): the score of
// rebuild_fast_split on the totals.
int rebuild_group_splits(int n, const int64_t* K, const int64_t* h_in, const int64_t* h_out) {
    int64_t tiles = 0, kmin = K[0];
    double ops = 0.0, outs = 0.0;
    for (int i = 0; i < n; ++i) {
        tiles += (h_in[i] / 256) * (h_out[i] / 256);
        ops += (double)K[i] * (h_in[i] + h_out[i]) * 2.0;
        outs += (double)h_in[i] * h_out[i] * 4.0;
        if (K[i] < kmin) kmin = K[i];
    }
    int best = 1;
    double best_score = -1.0;
    for (int s = 1; s <= 64; ++s) {
        if (s > 1 && kmin / s < 1024) break;
        const int64_t wg = tiles * s;
        const double eff = (double)wg / (double)(ceil_div(wg, 256) * 256);
        const double extra = s > 1 ? (2.0 * s + 1.0) * outs : 0.0;
        const double score = eff / (1.0 + extra / ops);
        if (score > best_score * 1.02) {
            best_score = score;
            best = s;
        }
    }
    return best;
}

SplitPlan rebuild_group_plan(int64_t K, int splits) {
    SplitPlan sp;
    sp.chunk = (int64_t)align_up((size_t)ceil_div(K, splits), rb::BK);
    sp.splits = (int)ceil_div(K, sp.chunk);
    return sp;
}

// n products (every one passes rebuild_group_ok; sp[i] from rebuild_group_plan) in launches of up to
// rb::MAX_JOBS; a product with sp[i].splits > 1 goes through slabs[i] and reduce_slabs.
dad_status launch_rebuild_group(int n, const void* const* L, const void* const* R, float* const* G, const int64_t* K,
                                const int64_t* h_in, const int64_t* h_out, const SplitPlan* sp, float* const* slabs,
                                hipStream_t s) {
    const int lds = rb::DMA_STAGES * 2 * rb::BK * 256 * 2;
    for (int first = 0; first < n; first += rb::MAX_JOBS) {
        const int cnt = n - first < rb::MAX_JOBS ? n - first : rb::MAX_JOBS;
        RebuildJobs tb;
        int64_t blocks = 0;
        bool ragged = false;
        for (int i = 0; i < rb::MAX_JOBS; ++i) {
            if (i >= cnt) {
                tb.first_block[i] = 0x7fffffff;
                tb.j[i] = RebuildJob{};
                continue;
            }
            const int k = first + i;
            RebuildJob& jb = tb.j[i];
            jb.L = static_cast<const bf16_t*>(L[k]);
            jb.R = static_cast<const bf16_t*>(R[k]);
            jb.out = sp[k].splits == 1 ? G[k] : slabs[k];
            jb.K = K[k];
            ragged |= K[k] % rb::BK != 0;
            jb.chunk = sp[k].chunk;
            jb.h_in = (int)h_in[k];
            jb.h_out = (int)h_out[k];
            jb.tiles_m = (int)(h_in[k] / 256);
            jb.tiles_n = (int)(h_out[k] / 256);
            tb.first_block[i] = (int)blocks;
            blocks += (int64_t)jb.tiles_m * jb.tiles_n * sp[k].splits;
            if (blocks > ((int64_t)1 << 30)) return DAD_ERR_SHAPE;
        }
        {
            ProfScope prof(KID_REBUILD_BF16_DMA, s);
            if (ragged)
                hipLaunchKernelGGL((k_rebuild_bf16_dma_jobs<256, 2, 4, true>), dim3((unsigned)blocks), dim3(512), lds, s, tb, (int)blocks);
            else
                hipLaunchKernelGGL((k_rebuild_bf16_dma_jobs<256, 2, 4, false>), dim3((unsigned)blocks), dim3(512), lds, s, tb, (int)blocks);
        }
        DAD_LAUNCH_CHECK();
    }
    SumJob sums[MAX_JOBS];
    int m = 0;
    for (int i = 0; i < n; ++i) {
        if (sp[i].splits > 1) sums[m++] = SumJob{slabs[i], G[i], nullptr, h_in[i] * h_out[i], sp[i].splits};
        if (m < MAX_JOBS && i + 1 < n) continue;
        const dad_status rc = reduce_slabs(sums, m, s);
        if (rc != DAD_OK) return rc;
        m = 0;
    }
    return DAD_OK;
}

// n products, each by its own plan (the bits are those of a call of its own) and with its slabs from G on, in as few launches as their
// kernels allow.
dad_status launch_rebuild_own(const OwnProduct* jobs, int n, dad_dtype dt, hipStream_t s) {
    if (n == 1 && dt == DAD_BF16) return launch_rebuild(jobs[0].L, jobs[0].R, jobs[0].K, jobs[0].h_in, jobs[0].h_out, dt, jobs[0].G, jobs[0].G, jobs[0].rb, s);
    if (n > MAX_JOBS) return DAD_ERR_SHAPE;
    if (dt == DAD_F32) {
        const void *L[MAX_JOBS], *R[MAX_JOBS];
        float* G[MAX_JOBS];
        int64_t K[MAX_JOBS], hi[MAX_JOBS], ho[MAX_JOBS];
        SplitPlan sp[MAX_JOBS];
        for (int i = 0; i < n; ++i) L[i] = jobs[i].L, R[i] = jobs[i].R, G[i] = jobs[i].G, K[i] = jobs[i].K, hi[i] = jobs[i].h_in, ho[i] = jobs[i].h_out, sp[i] = jobs[i].rb.split;
        return launch_rebuild_f32(n, L, R, G, K, hi, ho, sp, G, s, true);
    }
    constexpr int lds256 = rb::DMA_STAGES * 2 * rb::BK * 256 * 2, lds128 = rb::DMA_STAGES * 2 * rb::BK * 128 * 2;
    // 256-tiles, 128-tiles, any shape; of the first two, K of whole stages in one sum, and others
    auto kind = [&](const OwnProduct& j) { return j.rb.tile == 0 ? 4 : (j.rb.tile == 128 ? 2 : 0) + (j.rb.fine || j.K % rb::BK != 0); };
    SumJob sums[MAX_JOBS];
    int nsum = 0;
    for (int i = 0; i < n; ++i)
        if (jobs[i].rb.split.splits > 1) sums[nsum++] = SumJob{jobs[i].G, jobs[i].G, nullptr, jobs[i].h_in * jobs[i].h_out, jobs[i].rb.split.splits};
    for (int which = 0; which < 5; ++which) {
        int of[MAX_JOBS], c = 0;
        for (int i = 0; i < n; ++i)
            if (kind(jobs[i]) == which) {
                int at = c++;  // longest workgroups first
                for (; at > 0 && jobs[of[at - 1]].rb.split.chunk < jobs[i].rb.split.chunk; --at) of[at] = of[at - 1];
                of[at] = i;
            }
        for (int first = 0; first < c; first += rb::MAX_JOBS) {
            RebuildJobs tb;
            int64_t per = 0;  // workgroups of an XCD
            for (int i = 0; i < rb::MAX_JOBS; ++i) {
                if (first + i >= c) {
                    tb.first_block[i] = 0x7fffffff;
                    tb.j[i] = RebuildJob{};
                    continue;
                }
                const OwnProduct& j = jobs[of[first + i]];
                const int tile = j.rb.tile ? j.rb.tile : ra::TILE;
                const int64_t tm = ceil_div(j.h_in, tile), tn = ceil_div(j.h_out, tile), total = tm * tn * j.rb.split.splits;
                tb.first_block[i] = (int)per;
                per += ceil_div(total, 8);
                if (per > (int64_t)1 << 27) return DAD_ERR_SHAPE;
                tb.j[i] = RebuildJob{static_cast<const bf16_t*>(j.L), static_cast<const bf16_t*>(j.R), j.G, j.K, j.rb.split.chunk,
                                     (int)j.h_in, (int)j.h_out, (int)tm, (int)tn, (int)total};
            }
            const dim3 grid((unsigned)(8 * per));
            ProfScope prof(which == 4 ? KID_REBUILD_BF16 : KID_REBUILD_BF16_DMA, s);
            if (which == 0)
                hipLaunchKernelGGL((k_rebuild_bf16_dma_own<256, 2, 4, false>), grid, dim3(512), lds256, s, tb);
            else if (which == 1)
                hipLaunchKernelGGL((k_rebuild_bf16_dma_own<256, 2, 4, true>), grid, dim3(512), lds256, s, tb);
            else if (which == 2)
                hipLaunchKernelGGL((k_rebuild_bf16_dma_own<128, 2, 2, false>), grid, dim3(256), lds128, s, tb);
            else if (which == 3)
                hipLaunchKernelGGL((k_rebuild_bf16_dma_own<128, 2, 2, true>), grid, dim3(256), lds128, s, tb);
            else
                hipLaunchKernelGGL(k_rebuild_bf16_own, grid, dim3(ra::THREADS), ra::LDS, s, tb);
            DAD_LAUNCH_CHECK();
        }
    }
    return reduce_slabs(sums, nsum, s);
}

template <int T, int WM, int WN>
static dad_status prepare_dma() {
    constexpr int lds = rb::DMA_STAGES * 2 * rb::BK * T * 2;
    DAD_HIP_TRY(set_max_lds((k_rebuild_bf16_dma<T, WM, WN, RowBlocks, true>), lds));
    DAD_HIP_TRY(set_max_lds((k_rebuild_bf16_dma<T, WM, WN, const bf16_t*, false>), lds));
    DAD_HIP_TRY(set_max_lds((k_rebuild_bf16_dma<T, WM, WN, const bf16_t*, true>), lds));
    DAD_HIP_TRY(set_max_lds((k_rebuild_bf16_dma_own<T, WM, WN, false>), lds));
    DAD_HIP_TRY(set_max_lds((k_rebuild_bf16_dma_own<T, WM, WN, true>), lds));
    return DAD_OK;
}

dad_status rebuild_prepare_device() {
    constexpr int lds = rb::DMA_STAGES * 2 * rb::BK * 256 * 2;
    DAD_HIP_TRY(set_max_lds((k_rebuild_bf16_dma_jobs<256, 2, 4, false>), lds));
    DAD_HIP_TRY(set_max_lds((k_rebuild_bf16_dma_jobs<256, 2, 4, true>), lds));
    const dad_status rc = prepare_dma<256, 2, 4>();
    return rc != DAD_OK ? rc : prepare_dma<128, 2, 2>();
}

}  // namespace dad
