// Gradient rebuild G = L^T R (Eq. 4) for fp32 operands on the fp32 matrix instruction: the full gradient of
// the fp32 workloads (K = N) and the rank-r gradient P G^T of every workload (K = r; the sites' local
// rebuild of Algorithm 1).
//
// A wave owns a 64 x 64 tile of G and loads its operands straight from memory into the registers they are
// multiplied from: lane l takes four neighbouring columns 4 (l % 16) .. of K rows 4 (l / 16) .. + 3, 16 bytes at any
// float alignment, of each factor.  Column e of the lane is then operand e of v_mfma_f32_16x16x4_f32 (row l % 16,
// contraction l / 16), so the 4 x 4 products of a row quad cover the tile with its rows and columns interleaved
// by four, and a lane's results are four consecutive columns of G: 16-byte stores, a quarter wave a 256-byte piece
// of a row.  There is no LDS staging and no barrier in the contraction; 16 K rows (8 loads) per step, two steps in
// flight.  One wave per SIMD with its operands that far ahead keeps the matrix instruction busy (124 of its 130 TF from
// L2), and a second one only takes its lines: 70 TF, as the waves drift apart and each reads the L2 past the other.
// So a workgroup of four waves asks for the whole LDS of a compute unit, and the rest run in rounds; where the tiles
// are few for that, the waves of a workgroup split K and are summed through LDS in wave order, and only a long K goes
// through slabs and a second launch.
// What bounds it: the matrix instruction for K = N, the write of G for K = r.
// 2048 x 2048, K = 4096: 335 us with workgroups packed, 280 us so (123 TF); K = 1024, 784 x 1024 and 1024 x 1024 and
// 1024 x 10 in one call: 89 us on the LDS-staged kernel this replaced, 46 us.
// Edges: a lane whose columns would run past the last one is moved back to h - 4 (it computes and stores the same
// values as the lane that owns them), rows beyond K repeat row K - 1 with both operands masked to
// zero (an infinity in that row of one of them would make a NaN of the other's zero).
#include "dad_internal.h"

namespace dad {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef f32x4 f32x4_b4 __attribute__((aligned(4)));

namespace rf {
constexpr int NW = 4;           // waves per workgroup, one to a SIMD
constexpr int BK = 16;          // K rows per step
constexpr int MAX_JOBS = 32;
}  // namespace rf

struct alignas(64) RebuildF32Job {
    const float* L;
    const float* R;
    float* out;        // G, or the first of `splits` slabs of h_in * h_out floats
    int64_t K, chunk;  // chunk = K rows per slab, a multiple of 16 unless splits == 1
    int h_in, h_out, ks, splits;  // ks: waves that share a tile
    int wg;                       // workgroups
    int fold;                     // rounds of three steps per wave that are summed before they are added to the rest
};

// The tiles of a workgroup (NW / ks of them) form a block, so that they share operand lines in the L1.
__host__ __device__ inline int rf_block_m(int ks) { return ks == 1 ? 2 : 1; }
__host__ __device__ inline int rf_block_n(int ks) { return rf::NW / ks / rf_block_m(ks); }

// SHORT: less than eight steps (K = r, mostly).  What counts is that the loads, products and stores of several waves of a SIMD
// overlap, so the instance keeps two steps and no second accumulator: 163 registers, three waves to a SIMD.  32 products of
// 1024 x 1024 to 1024 x 4096, K = 32, in one launch: 160 us in the instance for a long K, 129 us so (LDS-staged kernel before 113).
// NT: non-temporal stores, for a launch whose results are larger than the Infinity Cache holds: 103 us there.  Smaller ones
// are left in the caches for whoever reads the gradients next.
template <int CAP, bool SHORT, bool NT>
__global__ __launch_bounds__(64 * rf::NW, SHORT ? 3 : 1) void k_rebuild_f32_mfma(JobTable<RebuildF32Job, CAP> tb) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    f32x4 (*red)[4][64] = reinterpret_cast<f32x4 (*)[4][64]>(smem);
    const RebuildF32Job& jb = tb.j[blockIdx.y];
    if ((int)blockIdx.x >= jb.wg) return;
    const int h_in = jb.h_in, h_out = jb.h_out, ks = jb.ks;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int kp = wave % ks, tile = wave / ks, bm = rf_block_m(ks), bn = rf_block_n(ks);
    const int wg_n = (h_out + 64 * bn - 1) / (64 * bn), wg_m = (h_in + 64 * bm - 1) / (64 * bm), per = wg_n * wg_m;
    // Workgroups go to the eight XCDs round-robin: those of one XCD take neighbouring tiles, whose operands they
    // share in its L2.
    int id = (int)blockIdx.x;
    {
        const int share = jb.wg >> 3, off = (int)(blockIdx.y * gridDim.x) & 7;
        if (id < share << 3) id = ((id + off) & 7) * share + (id >> 3);
    }
    const int split = id / per, at = id - split * per;
    const int p0 = ((at / wg_n) * bm + tile / bn) * 64, q0 = ((at % wg_n) * bn + tile % bn) * 64;
    const int c = lane & 15, q = lane >> 4;
    const int pc = p0 + 4 * c < h_in - 4 ? p0 + 4 * c : h_in - 4, qc = q0 + 4 * c < h_out - 4 ? q0 + 4 * c : h_out - 4;
    const int64_t kbeg = (int64_t)split * jb.chunk;
    const int64_t kend = kbeg + jb.chunk < jb.K ? kbeg + jb.chunk : jb.K;
    const int nb = (int)((kend - kbeg + rf::BK - 1) / rf::BK);
    const bool idle = p0 >= h_in || q0 >= h_out;  // a tile of the block outside the matrix

    constexpr int SETS = SHORT ? 2 : 3;
    f32x4 x[SETS][4], y[SETS][4];
    auto load = [&](auto set_c, int b) {
        constexpr int set = decltype(set_c)::value;
        const int64_t k0 = kbeg + (int64_t)b * rf::BK;
        const int lim = kend - 1 - k0 < rf::BK ? (int)(kend - 1 - k0) : rf::BK - 1;
        const float* l = jb.L + k0 * h_in;
        const float* r = jb.R + k0 * h_out;
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const int row = 4 * q + s, rc = row < lim ? row : lim;
            x[set][s] = *reinterpret_cast<const f32x4_b4*>(l + (uint32_t)rc * (uint32_t)h_in + pc);
            y[set][s] = *reinterpret_cast<const f32x4_b4*>(r + (uint32_t)rc * (uint32_t)h_out + qc);
        }
    };
    // The matrix instructions sum `fold` rounds of three steps (four: 192 K rows), which are then added to the rest: one running
    // sum over a wave's share of K rounds at full height with every instruction (2048 x 2304 x 756, error against fp64:
    // 5.7e-7 with one sum, 2.5e-7 so, the LDS-staged kernel before 4.7e-7; 4096 x 2048 x 2048: 274 -> 283 us, 384 rows 278 us
    // but 2560 x 403 x 977 then at 2.3e-7, before 2.1e-7).
    f32x4 acc[4][4], more[SHORT ? 1 : 4][4];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
            if constexpr (!SHORT) more[a][b] = acc[a][b];
        }
    const int fold_at = jb.fold;
    auto fold = [&]() {
        if constexpr (!SHORT) {
#pragma unroll
            for (int a = 0; a < 4; ++a)
#pragma unroll
                for (int b = 0; b < 4; ++b) {
                    more[a][b] += acc[a][b];
                    acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
                }
        }
    };
    auto compute = [&](auto set_c, int b) {
        constexpr int set = decltype(set_c)::value;
        const int64_t left = kend - kbeg - (int64_t)b * rf::BK;
        if (left < rf::BK) {
#pragma unroll
            for (int s = 0; s < 4; ++s)
                if (4 * q + s >= left) x[set][s] = y[set][s] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int s = 0; s < 4; ++s)
#pragma unroll
            for (int a = 0; a < 4; ++a)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    acc[a][e] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[set][s][a], y[set][s][e], acc[a][e], 0, 0, 0);
    };
    // loads are unconditional (a step beyond the last repeats it): the waits before a step's arithmetic
    // leave the next step in flight
    const std::integral_constant<int, 0> s0;
    const std::integral_constant<int, 1> s1;
    const std::integral_constant<int, SETS - 1> s2;
    if (SHORT) {
        if (!idle && kp < nb) {
            load(s0, kp);
            for (int b = kp; b < nb; b += 2 * ks) {
                if (b + ks < nb) load(s1, b + ks);
                __builtin_amdgcn_sched_barrier(0);
                compute(s0, b);
                __builtin_amdgcn_sched_barrier(0);
                if (b + 2 * ks < nb) load(s0, b + 2 * ks);
                __builtin_amdgcn_sched_barrier(0);
                if (b + ks < nb) compute(s1, b + ks);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    } else if (!idle && kp < nb) {
        auto at_most = [&](int b) { return b < nb ? b : nb - 1; };
        load(s0, kp);
        load(s1, at_most(kp + ks));
        int round = 0;
        for (int b = kp; b < nb; b += 3 * ks) {
            if (++round > fold_at) {
                fold();
                round = 1;
            }
            load(s2, at_most(b + 2 * ks));
            __builtin_amdgcn_sched_barrier(0);
            compute(s0, b);
            __builtin_amdgcn_sched_barrier(0);
            load(s0, at_most(b + 3 * ks));
            __builtin_amdgcn_sched_barrier(0);
            if (b + ks < nb) compute(s1, b + ks);
            __builtin_amdgcn_sched_barrier(0);
            load(s1, at_most(b + 4 * ks));
            __builtin_amdgcn_sched_barrier(0);
            if (b + 2 * ks < nb) compute(s2, b + 2 * ks);
            __builtin_amdgcn_sched_barrier(0);
        }
    }

    fold();
    f32x4 (&sum)[4][4] = [&]() -> f32x4 (&)[4][4] {
        if constexpr (SHORT) return acc;
        else return more;
    }();

    // sum[a][e][v]: row p0 + 16 q + 4 v + a, column q0 + 4 c + e.  A lane's row of a tile that was moved back:
    // its operand columns are pc .. pc + 3, i.e. rows indexed by the lane that holds them.
    float* o = jb.out + (int64_t)split * h_in * h_out;
    auto store = [&](int a, int v, f32x4 g) {
        const int i = 4 * q + v;  // row index of the matrix instruction: the lane i of the operand
        const int p = (p0 + 4 * i < h_in - 4 ? p0 + 4 * i : h_in - 4) + a;
        f32x4_b4* const at = reinterpret_cast<f32x4_b4*>(o + (int64_t)p * h_out + qc);
        if (NT)
            __builtin_nontemporal_store(g, at);
        else
            *at = g;
    };
    if (ks == 1) {
        if (idle) return;
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int v = 0; v < 4; ++v) store(a, v, f32x4{sum[a][0][v], sum[a][1][v], sum[a][2][v], sum[a][3][v]});
        return;
    }
#pragma unroll
    for (int a = 0; a < 4; ++a) {
        if (a) __syncthreads();
#pragma unroll
        for (int v = 0; v < 4; ++v) red[wave][v][lane] = f32x4{sum[a][0][v], sum[a][1][v], sum[a][2][v], sum[a][3][v]};
        __syncthreads();
        for (int v = kp; v < 4; v += ks) {
            f32x4 g = red[tile * ks][v][lane];
            for (int w = 1; w < ks; ++w) g += red[tile * ks + w][v][lane];
            if (!idle) store(a, v, g);
        }
    }
}

// One workgroup to a compute unit, in rounds over the chip's 256.  A wave's step costs about a microsecond, a round
// about five more (first loads, sum of the waves, store), slabs a launch and their way through memory.
static int64_t rf_groups(int64_t h_in, int64_t h_out, int ks) {
    return ceil_div(h_in, 64 * rf_block_m(ks)) * ceil_div(h_out, 64 * rf_block_n(ks));
}
static int64_t rf_cost(int64_t groups, int64_t steps, int ks, int64_t splits) {
    return ceil_div(groups * splits, CU_COUNT) * (ceil_div(steps, ks * splits) + 5);
}

// Waves of a tile and slabs of one product, by its own sizes alone: a product of a group gives the bits of a single call.
// Slabs of more than 64 MB have to gain 2 %: for the last percent a tall product would ask for hundreds of megabytes
// (97792 x 2432 x 874: 196 MB for 23 slabs, 51 MB for 6, 3.53 and 3.65 ms).
static SplitPlan rf_plan(int64_t K, int64_t h_in, int64_t h_out, int* waves) {
    const int64_t steps = ceil_div(K, rf::BK);
    struct { int64_t cost = INT64_MAX, splits = 1; int ks = 1; } best[2];  // slabs of up to 64 MB, and of more
    for (int ks = 1; ks <= rf::NW; ks *= 2)
        for (int64_t w = 1; w <= 64 && (w == 1 || w * ks * 8 <= steps); ++w) {
            const int64_t slabs = w == 1 ? 0 : 5 + (2 * w + 1) * h_in * h_out / 1000000;  // 4 bytes at 4 TB/s
            const int64_t cost = rf_cost(rf_groups(h_in, h_out, ks), steps, ks, w) + slabs;
            auto& b = best[w > 1 && w * h_in * h_out * 4 > (int64_t)64 << 20];
            if (cost < b.cost) b.cost = cost, b.splits = w, b.ks = ks;
        }
    const auto& b = best[best[1].cost < INT64_MAX && best[1].cost * 50 < best[0].cost * 49];
    const int64_t splits = b.splits;
    *waves = b.ks;
    SplitPlan sp;
    sp.chunk = splits == 1 ? K : (int64_t)align_up((size_t)ceil_div(K, splits), rf::BK);
    sp.splits = (int)ceil_div(K, sp.chunk);
    return sp;
}

// A product narrower than one 16-byte load stays on the guarded kernel.
bool rebuild_f32_ok(int64_t h_in, int64_t h_out) { return h_in >= 4 && h_out >= 4; }

SplitPlan rebuild_f32_split(int64_t K, int64_t h_in, int64_t h_out) {
    int ks;
    return rf_plan(K, h_in, h_out, &ks);
}

// As fitted to 200 products on the way to a reduction.
ProductTime rebuild_f32_time(int64_t K, int64_t h_in, int64_t h_out) {
    int ks;
    const SplitPlan sp = rf_plan(K, h_in, h_out, &ks);
    const int64_t groups = rf_groups(h_in, h_out, ks), steps = ceil_div(K, rf::BK);
    const double slabs = sp.splits == 1 ? 0.0 : (2.0 * sp.splits + 1.0) * h_in * h_out * 1e-6;
    const double wg = 5.0 + (double)ceil_div(steps, (int64_t)ks * sp.splits);
    return ProductTime{0.9 * ((sp.splits == 1 ? 0.0 : 5.0) + slabs + (double)rf_cost(groups, steps, ks, sp.splits)),
                       0.9 * (slabs + wg * (double)(groups * sp.splits) / CU_COUNT)};
}

// Launches n jobs (G_i = L_i^T R_i, each with its own split plan; a job with splits > 1 writes slabs
// at slabs[i] and is summed by reduce_slabs afterwards) in as few launches as the job table allows.
dad_status launch_rebuild_f32(int n, const void* const* L, const void* const* R, float* const* G, const int64_t* K,
                              const int64_t* h_in, const int64_t* h_out, const SplitPlan* sp, float* const* slabs,
                              hipStream_t s, bool fine) {
    for (int first = 0; first < n; first += rf::MAX_JOBS) {
        const int cnt = n - first < rf::MAX_JOBS ? n - first : rf::MAX_JOBS;
        RebuildF32Job jobs[rf::MAX_JOBS];
        SumJob sums[rf::MAX_JOBS];
        int most = 0, nsum = 0, nj = 0;
        int64_t longest = 0;  // steps of a slab
        double bytes = 0.0;   // of the results
        for (int i = first; i < first + cnt; ++i) {
            if (!rebuild_f32_ok(h_in[i], h_out[i])) {
                const dad_status rc = gen_rebuild(L[i], R[i], K[i], h_in[i], h_out[i], DAD_F32, G[i], slabs[i], sp[i], s);
                if (rc != DAD_OK) return rc;
                continue;
            }
            RebuildF32Job& jb = jobs[nj++];
            rf_plan(K[i], h_in[i], h_out[i], &jb.ks);
            jb.L = static_cast<const float*>(L[i]);
            jb.R = static_cast<const float*>(R[i]);
            jb.out = sp[i].splits == 1 ? G[i] : slabs[i];
            jb.K = K[i];
            jb.chunk = sp[i].chunk;
            jb.h_in = (int)h_in[i];
            jb.h_out = (int)h_out[i];
            jb.splits = sp[i].splits;
            const int64_t wg = rf_groups(h_in[i], h_out[i], jb.ks) * sp[i].splits;
            if (wg > (int64_t)1 << 30) return DAD_ERR_SHAPE;
            jb.wg = (int)wg;
            jb.fold = fine && ceil_div(jb.chunk, rf::BK) >= 8 ? 1 : 4;  // shorter ones have the bits of the instance for them
            if (jb.wg > most) most = jb.wg;
            if (ceil_div(jb.chunk, rf::BK) > longest) longest = ceil_div(jb.chunk, rf::BK);
            bytes += 4.0 * h_in[i] * h_out[i];
            if (sp[i].splits > 1) sums[nsum++] = SumJob{slabs[i], G[i], nullptr, h_in[i] * h_out[i], sp[i].splits};
        }
        if (nj) {
            ProfScope prof(KID_REBUILD_F32, s);
            // a short contraction is all first loads and stores: those overlap between workgroups of a compute unit
            const dim3 grid((unsigned)most, (unsigned)nj), block(64 * rf::NW);
            const auto launch = [&](auto tb, auto cap) {
                constexpr int CAP = decltype(cap)::value, LDS = rf::NW * 4 * 64 * 16;
                if (longest >= 8)
                    hipLaunchKernelGGL((k_rebuild_f32_mfma<CAP, false, false>), grid, block, CU_LDS, s, tb);
                else if (bytes > 200.0 * (1 << 20))
                    hipLaunchKernelGGL((k_rebuild_f32_mfma<CAP, true, true>), grid, block, LDS, s, tb);
                else
                    hipLaunchKernelGGL((k_rebuild_f32_mfma<CAP, true, false>), grid, block, LDS, s, tb);
            };
            if (nj <= 4)
                launch_jobs<4>(jobs, nj, launch);
            else
                launch_jobs<rf::MAX_JOBS>(jobs, nj, launch);
        }
        DAD_LAUNCH_CHECK();
        if (nsum) {
            const dad_status rc = reduce_slabs(sums, nsum, s);
            if (rc != DAD_OK) return rc;
        }
    }
    return DAD_OK;
}

dad_status rebuild_f32_prepare_device() {
    DAD_HIP_TRY(set_max_lds((k_rebuild_f32_mfma<1, false, false>), CU_LDS));
    DAD_HIP_TRY(set_max_lds((k_rebuild_f32_mfma<4, false, false>), CU_LDS));
    DAD_HIP_TRY(set_max_lds((k_rebuild_f32_mfma<rf::MAX_JOBS, false, false>), CU_LDS));
    return DAD_OK;
}

}  // namespace dad
