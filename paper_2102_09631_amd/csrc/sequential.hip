// Algorithm 2 as printed, one singular pair at a time with peeling (Section 3.3.1, Eq. 5-7), on top
// of the thin contraction kernels.  Component j iterates
//     g <- normalise( M^T M g - sum_{i<j} sigma_i^2 g_i (g_i^T g) )          n_iter times,
// then v = Delta g, p = A^T v, sigma_j = ||p|| (= sqrt(v^T A A^T v)), q_j = p / sigma_j, and the
// pair (q_j, sigma_j g_j) is kept.  The peeled term is the deflation of M^T M by the pairs already
// found (the printed Q (G^T g) mixes vectors of two lengths); with sG_i = sigma_i g_i it is
// sum_i sG_i (sG_i^T g).  Every thin pass is HBM bound and costs the same for one column as for 32,
// so this route costs r times the block form; it exists because it is the paper's own recurrence.
#include "dad_internal.h"

#include <type_traits>

namespace dad {

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
    return v;  // lane 0 holds the sum
}

// Sum over the 1024 threads of the workgroup; every thread gets the result.
__device__ __forceinline__ double block_sum(double v, double* red) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    v = wave_sum(v);
    __syncthreads();
    if (lane == 0) red[wave] = v;
    __syncthreads();
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < 16; ++w) s += red[w];
    return s;
}

// Control words of a call, in the 256-byte workspace header (cleared by the first launch):
//   int 0  numeric flag            int 1  skip: the running component needs no further application
//   int 2  done: no further component is wanted (the thin launches that follow return at once)
//   byte 128: double sigma_0
// In the adaptive mode (theta >= 0; Algorithm 2's stop test and the effective rank of Section 3.3.1)
// the found vectors are projected out of the start vector and of every iterate (the projector form of
// Eq. 7's peel); with theta < 0 the peel is the subtraction sum_i sigma_i^2 g_i (g_i . g) and the counts
// are fixed.
constexpr int SEQ_SKIP = 1, SEQ_DONE = 2;

// coef[i] = (sG_i . x) / (sG_i . sG_i) for i < j: the coefficient of the found direction i in x, times
// 1 / sigma_i (the rows of sGt are sigma_i g_i); one dot-product pair per wave.
__device__ __forceinline__ void seq_projection_coefs(const float* __restrict__ sGt, const float* __restrict__ x, int j,
                                                     int64_t h, double* coef) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    for (int i = wave; i < j; i += 16) {
        double sx = 0.0, ss = 0.0;
        for (int64_t k = lane; k < h; k += 64) {
            const double g = (double)sGt[(int64_t)i * h + k];
            sx += g * (double)x[k];
            ss += g * g;
        }
        sx = wave_sum(sx);
        ss = wave_sum(ss);
        if (lane == 0) coef[i] = ss > 0.0 ? sx / ss : 0.0;
    }
}

// Start of component j: g <- x / ||x||, in the adaptive mode after the found vectors are projected
// out of x.  The first launch of a call also clears the header.
__global__ __launch_bounds__(1024) void k_seq_start(const float* __restrict__ x, const float* __restrict__ sGt, int j,
                                                    float* __restrict__ g, int64_t h, int* __restrict__ hdr,
                                                    int clear_hdr, float theta, int* __restrict__ eff_rank,
                                                    int* __restrict__ iters) {
    __shared__ double red[16];
    __shared__ double coef[DAD_MAX_RANK];
    if (clear_hdr && threadIdx.x < 64) hdr[threadIdx.x] = 0;
    if (clear_hdr && threadIdx.x == 0 && eff_rank) *eff_rank = 0;
    __syncthreads();
    if (iters && threadIdx.x == 0) iters[j] = 0;
    if (hdr[SEQ_DONE]) {  // components are no longer wanted: everything up to the next start is skipped
        if (threadIdx.x == 0) hdr[SEQ_SKIP] = 1;
        return;
    }
    if (threadIdx.x == 0) hdr[SEQ_SKIP] = 0;
    const bool project = theta >= 0.f && j > 0;
    if (project) seq_projection_coefs(sGt, x, j, h, coef);
    __syncthreads();
    double ss = 0.0;
    for (int64_t k = threadIdx.x; k < h; k += 1024) {
        double v = (double)x[k];
        if (project)
            for (int i = 0; i < j; ++i) v -= coef[i] * (double)sGt[(int64_t)i * h + k];
        ss += v * v;
    }
    ss = block_sum(ss, red);
    if (!(ss > 0.0)) {
        if (threadIdx.x == 0) hdr[0] = 1;
        ss = 1.0;
    }
    const double inv = 1.0 / sqrt(ss);
    for (int64_t k = threadIdx.x; k < h; k += 1024) {
        double v = (double)x[k];
        if (project)
            for (int i = 0; i < j; ++i) v -= coef[i] * (double)sGt[(int64_t)i * h + k];
        g[k] = (float)(v * inv);
    }
}

// One application is done: y = M^T M g from the thin kernels.
//   theta < 0 : g <- normalise( y - sum_{i<j} sG_i (sG_i . g) )
//   theta >= 0: y <- y minus its components along the found vectors.  If nothing is left,
//               ||y|| < (theta sigma_0)^2, the gradient's rank is exhausted: done is set and component j
//               is dropped.  Otherwise g <- y / ||y||, and when the step from the old g (sign aligned)
//               is at most theta the remaining applications of this component are skipped.
__global__ __launch_bounds__(1024) void k_seq_update(const float* __restrict__ y, const float* __restrict__ sGt, int j,
                                                     float* __restrict__ g, int64_t h, int* __restrict__ hdr,
                                                     float theta, int* __restrict__ eff_rank, int* __restrict__ iters) {
    __shared__ double coef[DAD_MAX_RANK];
    __shared__ double red[16];
    if (hdr[SEQ_SKIP]) return;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const bool adaptive = theta >= 0.f;
    if (adaptive) {
        seq_projection_coefs(sGt, y, j, h, coef);
    } else {
        for (int i = wave; i < j; i += 16) {  // one dot product per wave
            double s = 0.0;
            for (int64_t k = lane; k < h; k += 64) s += (double)sGt[(int64_t)i * h + k] * (double)g[k];
            s = wave_sum(s);
            if (lane == 0) coef[i] = s;
        }
    }
    __syncthreads();
    if (!adaptive) {
        double ss = 0.0;
        for (int64_t k = threadIdx.x; k < h; k += 1024) {
            double v = (double)y[k];
            for (int i = 0; i < j; ++i) v -= coef[i] * (double)sGt[(int64_t)i * h + k];
            g[k] = (float)v;  // the old g is no longer needed: the dot products are done
            ss += v * v;
        }
        ss = block_sum(ss, red);
        if (!(ss > 0.0)) {  // nothing left in this direction (or NaN): latch and leave the vector finite
            if (threadIdx.x == 0) hdr[0] = 1;
            ss = 1.0;
        }
        const float inv = (float)(1.0 / sqrt(ss));
        for (int64_t k = threadIdx.x; k < h; k += 1024) g[k] *= inv;
        return;
    }
    double ss = 0.0, dot = 0.0;
    for (int64_t k = threadIdx.x; k < h; k += 1024) {
        double v = (double)y[k];
        for (int i = 0; i < j; ++i) v -= coef[i] * (double)sGt[(int64_t)i * h + k];
        ss += v * v;
        dot += v * (double)g[k];
    }
    ss = block_sum(ss, red);
    dot = block_sum(dot, red);
    if (threadIdx.x == 0 && iters) iters[j] += 1;
    if (j > 0) {
        const double s0 = *reinterpret_cast<const double*>(reinterpret_cast<const char*>(hdr) + 128);
        const double lim = (double)theta * s0;
        if (sqrt(ss) < lim * lim) {  // nothing left to iterate on
            if (threadIdx.x == 0) {
                hdr[SEQ_SKIP] = 1;
                hdr[SEQ_DONE] = 1;
                if (eff_rank) *eff_rank = j;
            }
            return;
        }
    }
    if (!(ss > 0.0)) {
        if (threadIdx.x == 0) hdr[0] = 1;
        ss = 1.0;
    }
    const double inv = 1.0 / sqrt(ss);
    const double sgn = dot < 0.0 ? -1.0 : 1.0;
    double step2 = 0.0;
    for (int64_t k = threadIdx.x; k < h; k += 1024) {
        double v = (double)y[k];
        for (int i = 0; i < j; ++i) v -= coef[i] * (double)sGt[(int64_t)i * h + k];
        const float gn = (float)(v * inv);
        const double d = sgn * (double)gn - (double)g[k];
        step2 += d * d;
        g[k] = gn;
    }
    step2 = block_sum(step2, red);
    if (threadIdx.x == 0 && sqrt(step2) <= (double)theta) hdr[SEQ_SKIP] = 1;
}

// sigma = ||p||, q = p / sigma, sG = sigma g.  Adaptive mode: a component with sigma < theta sigma_0 is
// dropped and ends the call's iteration; rows of dropped components are zero.
__global__ __launch_bounds__(1024) void k_seq_finish(const float* __restrict__ p, const float* __restrict__ g,
                                                     float* __restrict__ q_row, float* __restrict__ sg_row,
                                                     float* __restrict__ sigma_out, int64_t h_in, int64_t h_out,
                                                     int* __restrict__ hdr, int j, float theta,
                                                     int* __restrict__ eff_rank) {
    __shared__ double red[16];
    double* s0 = reinterpret_cast<double*>(reinterpret_cast<char*>(hdr) + 128);
    bool drop = hdr[SEQ_DONE] != 0;
    double sigma = 0.0;
    if (!drop) {
        double ss = 0.0;
        for (int64_t k = threadIdx.x; k < h_in; k += 1024) ss += (double)p[k] * (double)p[k];
        ss = block_sum(ss, red);
        sigma = sqrt(ss);
        if (theta >= 0.f && j > 0 && sigma < (double)theta * *s0) {
            drop = true;
            __syncthreads();  // every thread has read the flag and sigma_0
            if (threadIdx.x == 0) {
                hdr[SEQ_DONE] = 1;
                if (eff_rank) *eff_rank = j;
            }
        }
    }
    if (drop) {
        for (int64_t k = threadIdx.x; k < h_in; k += 1024) q_row[k] = 0.f;
        for (int64_t k = threadIdx.x; k < h_out; k += 1024) sg_row[k] = 0.f;
        if (sigma_out && threadIdx.x == 0) *sigma_out = 0.f;
        return;
    }
    if (!(sigma > 0.0)) {
        if (threadIdx.x == 0) hdr[0] = 1;
        sigma = 0.0;
    }
    const double inv = sigma > 0.0 ? 1.0 / sigma : 0.0;
    for (int64_t k = threadIdx.x; k < h_in; k += 1024) q_row[k] = (float)((double)p[k] * inv);
    for (int64_t k = threadIdx.x; k < h_out; k += 1024) sg_row[k] = (float)(sigma * (double)g[k]);
    if (threadIdx.x == 0) {
        if (sigma_out) *sigma_out = (float)sigma;
        if (j == 0) *s0 = sigma;
        if (eff_rank) *eff_rank = j + 1;
    }
}

// ------------------------------------------------------------------------------------------------
// The recurrence on M (fixed counts): one launch per application.  A row of M gives its part of M^T (M g) by itself,
// v = row . g and then v * row, so a workgroup keeps a few rows in registers for both products and leaves a slab of M^T M g.
// The next launch starts with what a launch of its own did before: every workgroup adds the slabs, subtracts the peel and
// normalises, all in fp64 and alike, while its rows of M are on their way.  One workgroup more than the rows need keeps the
// books: it ends the component before, forms the peel of the running vector for the next launch, and latches the status.
// What bounds it: latency (a launch, the slabs' round trip through the memory side, a barrier per batch of rows), which is why the slabs are
// few (SEQ_SLABS) and the threads are split into G groups that take slabs and rows in turn.
// A whole call, 768 x 768, N = 4096, 8 components, two applications: 72 launches beside those that make M, 434 us, with a launch per
// product, update, start and end; 25 and 200 us so (a launch 7 to 8 us).
// PAIR: two launches per application, where the workspace, which was sized for a launch per step, has no room for the slabs, or where M is
// long for 64 workgroups or its rows are wide (seq_slabs_win).  This one takes M g alone, with every unit, and k_thin_tn_direct M^T of that; the
// next one adds the slabs of that launch, which fit where they always were.  With two running vectors in turn in place of peels each
// workgroup forms the peel for itself.
// N = 64, 784 x 128, 4 components: 155 us with a launch per step, 119 so (79 with slabs); N = 4096, 3072 x 768, 8 components: 435, 310 (270);
// N = 300, 1024 x 4096, 16 components: 1507, 973 (1097); N = 32768, 16384 x 4096, 8 components: 6654, 5860 (8458).
// Rows wider than SEQ_ROW_MOST, and the adaptive mode (its stop test sits between an update and the next product), keep a launch per step.
// Column layout: thread c of a group holds columns at .. at + 3, at = min(4 c, h_out - 4); those of the thread before it count
// as zero in g and have the same values in both otherwise.
// ------------------------------------------------------------------------------------------------
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef f32x4 f32x4_b4 __attribute__((aligned(4)));

constexpr int SEQ_SLABS = 64;           // at most; each workgroup reads them all
constexpr int64_t SEQ_ROW_MOST = 4096;  // columns of one workgroup: 1024 threads of four
constexpr int SEQ_ROWS = 4;             // rows of a group in flight, twice
constexpr int SEQ_UNITS = CU_COUNT - 1;  // workgroups of rows of the PAIR form, one to a unit with the books

enum { SEQ_FIRST = 1, SEQ_LAST = 2 };  // the launch that starts a component, the one that ends its iteration

struct SeqProduct {
    const float* M;
    const float* x;       // start vector (first launch)
    const float* slabs;   // of the application before, `nslabs` of them
    const double* peel;   // and the peel of its vector
    const float* g_before;  // the running vector of the launch before (PAIR; first launch: of the component before)
    const float* p_before;  // M g of the component before (first launch)
    float* slabs_out;
    double* peel_out;
    float* p;             // M g (last launch; PAIR: every one, with zeros from h_in to h_pad)
    float* g;             // the running vector, as the last launch leaves it (PAIR: every one)
    float *Qt, *sGt, *sigma;
    int* hdr;
    int h_in, h_pad, h_out, j, blocks, batches, nslabs, mode, clear_hdr;
};

// Thread groups of a workgroup; their threads (whole waves).
static int seq_lanes(int64_t h_out) { return (int)align_up((size_t)ceil_div(h_out, 4), 64); }
static int seq_groups(int64_t h_out) {
    const int n = seq_lanes(h_out);
    return n <= 128 ? 8 : n <= 256 ? 4 : n <= 512 ? 2 : 1;
}
// Batches of rows of a workgroup, of at most `most` workgroups; their number.
static int seq_batches(int64_t h_in, int64_t h_out, int most) { return (int)ceil_div(h_in, (int64_t)SEQ_ROWS * seq_groups(h_out) * most); }
static int seq_blocks(int64_t h_in, int64_t h_out, int most) {
    return (int)ceil_div(h_in, (int64_t)SEQ_ROWS * seq_groups(h_out) * seq_batches(h_in, h_out, most));
}

// 64 workgroups read M at 1.7 TB/s (a batch of theirs, 4 MB, 2.4 us), against 5 to 6 TB/s of two launches on all units, and wide rows make
// wide slabs.  Whole calls, N = 4096, two applications, 4 and 16 components, slabs and PAIR: 8192 x 1024 (8 batches) 324 and 324, 1048 and 1063 us;
// 12288 x 1024 442 and 401, 1443 and 1292; 3072 x 2048 (6) 278 and 260, 906 and 879; 16384 x 512 (8) 292 and 330; 16384 x 256 (8) 225 and 245, 732 and 829;
// 24576 x 256 (12) 294 and 300; 24576 x 128 279 and 273.  Rows of one group: 768 x 2304 192 and 188, 686 and 736; 1024 x 2304 216 and 184, 750 and 694;
// 256 x 3072 167 and 160, 676 and 666; 768 x 3072 225 and 211, 797 and 826; 256 x 4096 202 and 176, 835 and 781; 1024 x 4096 308 and 245, 1100 and 983.
static bool seq_slabs_win(int64_t h_in, int64_t h_out) {
    const int64_t batches = seq_batches(h_in, h_out, SEQ_SLABS);
    return seq_groups(h_out) > 1 && batches <= 8 && batches * h_out <= 8192;
}

// v[i], i < 4, summed over the wave: lane l returns the sum of v[l & 3].
template <typename T> __device__ __forceinline__ T wave_sum4(const T (&v)[4]) {
    const int lane = threadIdx.x & 63;
    const bool b0 = lane & 1, b1 = lane & 2;
    // the lane keeps the values whose index ends in its own low bits, and hands the others over
    T a0 = (b0 ? v[1] : v[0]) + __shfl_xor(b0 ? v[0] : v[1], 1, 64);
    T a1 = (b0 ? v[3] : v[2]) + __shfl_xor(b0 ? v[2] : v[3], 1, 64);
    T s = (b1 ? a1 : a0) + __shfl_xor(b1 ? a0 : a1, 2, 64);
#pragma unroll
    for (int o = 4; o < 64; o <<= 1) s += __shfl_xor(s, o, 64);
    return s;
}

template <int G, bool PAIR>
__global__ __launch_bounds__(1024) void k_seq_product(const SeqProduct a) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    __shared__ double sums[2][16][4];  // per wave
    const int n = blockDim.x / G, grp = threadIdx.x / n, c = threadIdx.x - grp * n;  // n: threads of a group, whole waves
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, wpg = n >> 6, w0 = grp * wpg;
    const int h = a.h_out;
    const int at = 4 * c < h - 4 ? 4 * c : h - 4;
    bool own[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) own[e] = 4 * c < h && at + e >= 4 * c;
    const bool books = (int)blockIdx.x == a.blocks, first = a.mode & SEQ_FIRST, last = a.mode & SEQ_LAST;

    f32x4 m[2][SEQ_ROWS];
    auto row0 = [&](int b) { return (((int)blockIdx.x * a.batches + b) * G + grp) * SEQ_ROWS; };
    auto load = [&](auto set_c, int b) {
        constexpr int set = decltype(set_c)::value;
#pragma unroll
        for (int i = 0; i < SEQ_ROWS; ++i) {
            const int row = row0(b) + i;
            m[set][i] = *reinterpret_cast<const f32x4_b4*>(a.M + (int64_t)(row < a.h_in ? row : a.h_in - 1) * h + at);
        }
    };
    const std::integral_constant<int, 0> s0;
    const std::integral_constant<int, 1> s1;
    if (!books) load(s0, 0);

    // the vector: every group has all of it
    double v[4] = {0.0, 0.0, 0.0, 0.0};
    double(*red)[4] = reinterpret_cast<double(*)[4]>(smem);  // [threadIdx.x]
    // peel of x: sum over the found pairs of sG_i (sG_i . x), the groups taking four pairs at a time in turn; each group's part.  PAIR: nothing was
    // read from `sums` before
    auto peel_of = [&](const float(&x)[4], double(&z)[4]) {
#pragma unroll
        for (int e = 0; e < 4; ++e) z[e] = 0.0;
        for (int i0 = 0, turn = 0; i0 < a.j; i0 += 4 * G, turn ^= 1) {
            const int i1 = i0 + 4 * grp;
            f32x4 sg[4];
            double d[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) sg[u] = *reinterpret_cast<const f32x4_b4*>(a.sGt + (int64_t)(i1 + u < a.j ? i1 + u : 0) * h + at);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                d[u] = 0.0;
#pragma unroll
                for (int e = 0; e < 4; ++e) d[u] += (double)sg[u][e] * (double)x[e];
            }
            const double t = wave_sum4(d);
            if (turn == 0 && (!PAIR || i0 > 0)) __syncthreads();  // every reader of the buffer's last contents is done
            if (lane < 4) sums[turn][wave][lane] = t;
            __syncthreads();
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                double s = 0.0;
                for (int w = 0; w < wpg; ++w) s += sums[turn][w0 + w][u];
                if (i1 + u < a.j)
#pragma unroll
                    for (int e = 0; e < 4; ++e) z[e] += s * (double)sg[u][e];
            }
        }
    };
    if (first) {
        const f32x4 x = *reinterpret_cast<const f32x4_b4*>(a.x + at);
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = (double)x[e];
    } else {
        constexpr int P = G < 8 ? 16 : 8;  // slabs in flight: all of a group's from G = 4 on
        const float* src = a.slabs + at;
        auto slab = [&](int b) -> f32x4 { return *reinterpret_cast<const f32x4_b4*>(src + (int64_t)(b < a.nslabs ? b : a.nslabs - 1) * h); };
        double z[4];
        if constexpr (PAIR) {  // a few slabs, the first ones on their way during the peel; v is the group's part of both
            f32x4 t = slab(grp);
            float x[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) x[e] = own[e] ? a.g_before[at + e] : 0.f;
            peel_of(x, z);
            for (int b = grp; b < a.nslabs; b += G) {
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] += (double)t[e];
                if (b + G < a.nslabs) t = slab(b + G);
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] -= z[e];
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) z[e] = a.peel[at + e];
            for (int b = grp; b < a.nslabs; b += P * G) {
                f32x4 t[P];
#pragma unroll
                for (int u = 0; u < P; ++u) t[u] = slab(b + u * G);
#pragma unroll
                for (int u = 0; u < P; ++u)
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] += b + u * G < a.nslabs ? (double)t[u][e] : 0.0;
            }
        }
        if constexpr (G > 1) {
#pragma unroll
            for (int e = 0; e < 4; ++e) red[threadIdx.x][e] = v[e];
            __syncthreads();
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                v[e] = red[c][e];
#pragma unroll
                for (int q = 1; q < G; ++q) v[e] += red[q * n + c][e];
            }
        }
        if constexpr (!PAIR)
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] -= z[e];
        else if constexpr (G == 1)
            __syncthreads();  // the peel's sums have been read
    }
    double sq = 0.0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        v[e] = own[e] ? v[e] : 0.0;
        sq += v[e] * v[e];
    }
    sq = wave_sum(sq);
    if (lane == 0) sums[0][wave][0] = sq;
    if (books && a.clear_hdr && threadIdx.x < 64) a.hdr[threadIdx.x] = 0;
    __syncthreads();
    double ss = 0.0;
    for (int w = 0; w < wpg; ++w) ss += sums[0][w0 + w][0];
    const bool gone = !(ss > 0.0);  // nothing left in this direction (or NaN): latch and leave the vector finite
    if (books && gone && threadIdx.x == 0) a.hdr[0] = 1;
    const double inv = gone ? 1.0 : 1.0 / sqrt(ss);
    float g[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) g[e] = (float)(v[e] * inv);

    if (!books) {
        f32x4 y = {0.f, 0.f, 0.f, 0.f};
        auto rows = [&](auto set_c, int b) {
            constexpr int set = decltype(set_c)::value;
            float d[SEQ_ROWS];
#pragma unroll
            for (int i = 0; i < SEQ_ROWS; ++i) {
                d[i] = 0.f;
#pragma unroll
                for (int e = 0; e < 4; ++e) d[i] = fmaf(m[set][i][e], g[e], d[i]);
            }
            double t = wave_sum4(d);
            if (lane < 4) sums[(b + 1) & 1][wave][lane] = t;
            __syncthreads();
            const int r0 = row0(b);
#pragma unroll
            for (int i = 0; i < SEQ_ROWS; ++i) {
                double s = 0.0;
                for (int w = 0; w < wpg; ++w) s += sums[(b + 1) & 1][w0 + w][i];
                const float x = r0 + i < a.h_in ? (float)s : 0.f;
                if (PAIR || last) {
                    if (c == 0 && r0 + i < a.h_in) a.p[r0 + i] = x;
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) y[e] = fmaf(x, m[set][i][e], y[e]);
                }
            }
        };
        for (int b = 0; b < a.batches; b += 2) {
            if (b + 1 < a.batches) load(s1, b + 1);
            rows(s0, b);
            if (b + 1 < a.batches) {
                if (b + 2 < a.batches) load(s0, b + 2);
                rows(s1, b + 1);
            }
        }
        if (PAIR || last) return;
        f32x4* ysum = reinterpret_cast<f32x4*>(smem);
        if constexpr (G > 1) {
            ysum[threadIdx.x] = y;  // the sums over slabs were read before the barriers above
            __syncthreads();
#pragma unroll
            for (int q = 1; q < G; ++q)
                if (grp == 0) y += ysum[q * n + c];
        }
        if (grp == 0 && 4 * c < h) *reinterpret_cast<f32x4_b4*>(a.slabs_out + (int64_t)blockIdx.x * h + at) = y;
        return;
    }

    // the books
    if (PAIR && (int)threadIdx.x < a.h_pad - a.h_in) a.p[a.h_in + threadIdx.x] = 0.f;
    if (first && a.j > 0) {  // sigma = ||p||, q = p / sigma and sG = sigma g of the component before
        double t = 0.0;
        for (int k = threadIdx.x; k < a.h_in; k += blockDim.x) t += (double)a.p_before[k] * (double)a.p_before[k];
        t = wave_sum(t);
        if (lane == 0) sums[1][wave][0] = t;
        __syncthreads();
        double pp = 0.0;
        for (int w = 0; w < (int)blockDim.x >> 6; ++w) pp += sums[1][w][0];
        double sigma = sqrt(pp);
        if (!(sigma > 0.0)) {
            if (threadIdx.x == 0) a.hdr[0] = 1;
            sigma = 0.0;
        }
        const double is = sigma > 0.0 ? 1.0 / sigma : 0.0;
        float* q_row = a.Qt + (int64_t)(a.j - 1) * a.h_in;
        float* sg_row = a.sGt + (int64_t)(a.j - 1) * h;
        for (int k = threadIdx.x; k < a.h_in; k += blockDim.x) q_row[k] = (float)((double)a.p_before[k] * is);  // PAIR: in place
        for (int k = threadIdx.x; k < h; k += blockDim.x) sg_row[k] = (float)(sigma * (double)a.g_before[k]);
        if (a.sigma && threadIdx.x == 0) a.sigma[a.j - 1] = (float)sigma;
        __threadfence_block();
        __syncthreads();
    }
    if (PAIR || last) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (grp == 0 && own[e]) a.g[at + e] = g[e];
        return;
    }
    double z[4];
    peel_of(g, z);
    if constexpr (G > 1) {
        __syncthreads();
#pragma unroll
        for (int e = 0; e < 4; ++e) red[threadIdx.x][e] = z[e];
        __syncthreads();
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            z[e] = red[c][e];
#pragma unroll
            for (int q = 1; q < G; ++q) z[e] += red[q * n + c][e];
        }
    }
    if (grp == 0)
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (own[e]) a.peel_out[at + e] = z[e];
}

template <bool PAIR>
static dad_status seq_product(const SeqProduct& a, hipStream_t s) {
    const int groups = seq_groups(a.h_out), threads = groups * seq_lanes(a.h_out), lds = groups > 1 ? threads * 32 : 0;
    const dim3 grid((unsigned)a.blocks + 1);
    ProfScope prof(KID_SEQ_PRODUCT, s);
    switch (groups) {
        case 8: hipLaunchKernelGGL((k_seq_product<8, PAIR>), grid, dim3(threads), lds, s, a); break;
        case 4: hipLaunchKernelGGL((k_seq_product<4, PAIR>), grid, dim3(threads), lds, s, a); break;
        case 2: hipLaunchKernelGGL((k_seq_product<2, PAIR>), grid, dim3(threads), lds, s, a); break;
        default:
            if constexpr (!PAIR) return DAD_ERR_SHAPE;  // seq_slabs_win
            else hipLaunchKernelGGL((k_seq_product<1, PAIR>), grid, dim3(threads), lds, s, a);
    }
    DAD_LAUNCH_CHECK();
    return DAD_OK;
}

// The recurrence is a chain of short launches, and a product with M = A^T Delta is one of them where a product with
// the factors is two and a slab sum: M is made first wherever seq_dense_wins says so.  768 x 768, N = 4096, bf16, 8
// components: 624 us on the factors, 198 us on M (of which M 20 us).
// The workspace holds the layout of the route taken, products on the factors (c) or on the gradient (d), and behind
// it the running vector (h_out fp32).
struct SeqPlan {
    CompressPlan c;
    DensePlan d;
    size_t off_panel;
    size_t total;
    bool dense;        // some number of components is faster on the gradient: the workspace holds it
    bool fused;        // and a workgroup holds its rows: k_seq_product
    bool pair;         // two launches per application: faster, or no room for
    size_t slab_bytes, peel_bytes;  // those of one application, two of each over the slabs M was made from, which are done with by then
};

// The size query knows neither the components nor their applications; from 64 vectors' worth of products on nothing
// changes any more.
constexpr int64_t SEQ_MANY_PRODUCTS = 64 * 5;

static SeqPlan plan_sequential(int64_t N, int64_t h_in, int64_t h_out, dad_dtype dt) {
    SeqPlan p;
    const size_t vec = align_up((size_t)h_out * 4, 256);
    p.c = plan_factors(N, h_in, h_out, 1, dt);
    p.d = plan_dense(N, h_in, h_out, 1, dt);
    p.dense = dense_wins(N, h_in, h_out, dt, SEQ_MANY_PRODUCTS);
    const size_t factors = p.c.off_Yt + vec;  // nothing is orthonormalised: the layout ends with its Yt
    p.off_panel = p.dense && p.d.total > factors ? p.d.total : factors;
    p.fused = p.dense && h_out >= 4 && h_out <= SEQ_ROW_MOST;
    p.peel_bytes = align_up((size_t)h_out * 8, 256);
    p.slab_bytes = p.fused ? align_up((size_t)seq_blocks(h_in, h_out, SEQ_SLABS) * h_out * 4, 256) : 0;
    p.pair = !seq_slabs_win(h_in, h_out) || p.d.off_slabs + 2 * (p.slab_bytes + p.peel_bytes) > p.off_panel;
    p.total = p.off_panel + vec;
    return p;
}

// Whether a call whose workspace holds M makes it.  The adaptive mode asks for one component's first products for certain (dense_wins).
// Fixed counts, in microseconds: on the factors a product as in dense_wins and a vector launch at the start, the end and after each
// application; on M the launches of k_seq_product's two forms.  Of 424 shapes that were faster on M by this rule or one near it (128 to 40000 rows,
// widths 48 to 4500, 1 to 16 components, both types) none is slower on the route taken by 3 %; with the products alone counted, two launches each,
// and ragged bf16 products at 0.25e9 flops per us, 149 drawn shapes took 3 % more on average.  N = 4974, 3023 x 469, one component: 150 us on the
// factors, 79 on M.
static bool seq_dense_wins(const SeqPlan& p, int64_t N, int64_t h_in, int64_t h_out, dad_dtype dt, int r, int n_iter, bool adaptive) {
    if (!p.dense) return false;
    if (adaptive || !p.fused) return dense_wins(N, h_in, h_out, dt, adaptive ? 5 : (int64_t)r * (2 * (int64_t)n_iter + 1));
    const bool whole = N >= 256 && h_in % 128 == 0 && h_out % 128 == 0;
    const double rate = dt == DAD_F32 ? 0.8e8 : whole ? 0.8e9 : 0.4e9;  // flops per us
    const double h = (double)h_out, bytes = (double)h_in * h * 4.0, both = (double)N * (h_in + h) * elem_size(dt), n = n_iter;
    const double factors = r * ((2.0 * n + 1.0) * (8.0 + both / 5e6 + (N > 256 ? 2.5 : 0.0)) + (n + 2.0) * (4.0 + 1.2e-3 * h));
    const double pair = (n + 1.0) * (5.0 + 1e-3 * h + bytes / 5e6) + n * (5.0 + bytes / 5e6);
    const double slabs = (n + 1.0) * (4.0 + 2.2e-3 * h + bytes / 2.2e6);
    return 12.0 + 2.0 * N * h_in * h / rate + r * (p.pair ? pair : slabs) < 0.95 * factors;
}

}  // namespace dad

using namespace dad;

static bool seq_shape_ok(int64_t N, int64_t h_in, int64_t h_out, int r) {
    if (N < 1 || h_in < 1 || h_out < 1 || r < 1 || r > DAD_MAX_RANK) return false;
    if (r > N || r > h_in || r > h_out) return false;
    return N <= DAD_MAX_ROWS && h_in <= DAD_MAX_WIDTH && h_out <= DAD_MAX_WIDTH;
}

extern "C" size_t dad_compress_sequential_workspace_bytes(int64_t N, int64_t h_in, int64_t h_out, dad_dtype dt) {
    if ((dt != DAD_F32 && dt != DAD_BF16) || !seq_shape_ok(N, h_in, h_out, 1)) return 0;
    return plan_sequential(N, h_in, h_out, dt).total;
}

// The launches of the one-vector recurrence; theta < 0: fixed counts, subtraction peel.
static dad_status sequential_launch(const SeqPlan& p, const void* A, const void* D, int64_t N, int64_t h_in,
                                    int64_t h_out, dad_dtype dt, int r, int n_iter, float theta, const float* G0,
                                    float* Qt, float* sGt, float* sigma, int* eff_rank, int* iters, void* workspace,
                                    hipStream_t s) {
    char* ws = static_cast<char*>(workspace);
    const bool adaptive = theta >= 0.f;
    const bool dense = seq_dense_wins(p, N, h_in, h_out, dt, r, n_iter, adaptive);
    const CompressPlan& c = dense ? p.d.m : p.c;
    int* hdr = reinterpret_cast<int*>(ws + c.off_flag);
    void* V = ws + c.off_V;
    float* part = reinterpret_cast<float*>(ws + c.off_part);
    float* Ut = reinterpret_cast<float*>(ws + c.off_Ut);
    float* Yt = reinterpret_cast<float*>(ws + c.off_Yt);
    float* M = reinterpret_cast<float*>(ws + p.d.off_M);
    float* panel = reinterpret_cast<float*>(ws + p.off_panel);  // g
    // device-side stop flags the thin launches honour (adaptive mode only)
    const int* skip_iter = adaptive ? hdr + SEQ_SKIP : nullptr;
    const int* skip_done = adaptive ? hdr + SEQ_DONE : nullptr;
    dad_status rc;
#define DAD_TRY(expr)                           \
    do {                                        \
        if ((rc = (expr)) != DAD_OK) return rc; \
    } while (0)
    const int64_t rows = dense ? h_in : N;  // of the matrices the vectors are multiplied with
    const dad_dtype xt = dense ? DAD_F32 : dt;
    auto nn = [&](const void* X, const float* P, int64_t h, SplitPlan sp, const int* skip) {
        if (!c.direct) return gen_thin_nn(X, P, V, part, sp, rows, h, 1, xt, nullptr, s, skip);
        const NnJob j = {X, P, static_cast<float*>(V), part, nullptr, rows, (int)h, (short)sp.splits, xt == DAD_F32, 0, 0};
        return direct_nn(&j, 1, 1, s, skip);
    };
    auto tn = [&](const void* X, float* out, int64_t h, SplitPlan sp, const int* skip) {
        if (!c.direct) return gen_thin_tn(X, V, out, part, sp, rows, h, 1, xt, s, skip);
        const TnJob j = {X, static_cast<const float*>(V), sp.splits == 1 ? out : part, rows, sp.chunk, (int)h, sp.splits, xt == DAD_F32};
        const dad_status rc = direct_tn(&j, 1, 1, s, skip);
        return rc == DAD_OK && sp.splits > 1 ? reduce_slabs(part, out, h, sp.splits, s, nullptr, skip) : rc;
    };
    // y = M^T M g, and p = M g (in V on the gradient, in Ut on the factors)
    auto apply = [&]() {
        dad_status rc;
        if (dense) {
            DAD_TRY(nn(M, panel, h_out, c.nn_out, skip_iter));
            return tn(M, Yt, h_out, c.tn_out, skip_iter);
        }
        DAD_TRY(nn(D, panel, h_out, c.nn_out, skip_iter));  // v = Delta g
        DAD_TRY(tn(A, Ut, h_in, c.tn_in, skip_iter));       // u = A^T v
        DAD_TRY(nn(A, Ut, h_in, c.nn_in, skip_iter));       // w = A u
        return tn(D, Yt, h_out, c.tn_out, skip_iter);       // y = Delta^T w
    };
    auto last = [&]() {
        dad_status rc;
        DAD_TRY(nn(dense ? M : D, panel, h_out, c.nn_out, skip_done));
        return dense ? DAD_OK : tn(A, Ut, h_in, c.tn_in, skip_done);
    };
    const float* const p_vec = dense ? static_cast<const float*>(V) : Ut;
    if (dense) DAD_TRY(launch_rebuild(A, D, N, h_in, h_out, dt, M, reinterpret_cast<float*>(ws + p.d.off_slabs), p.d.rb, s));
    if (dense && p.fused && !adaptive) {
        SeqProduct a = {};
        char* const slabs = ws + p.d.off_slabs;
        char* const peels = slabs + 2 * p.slab_bytes;
        const int most = p.pair ? SEQ_UNITS : SEQ_SLABS;
        a.M = M, a.p = static_cast<float*>(V), a.g = panel, a.Qt = Qt, a.sGt = sGt, a.sigma = sigma, a.hdr = hdr;
        a.h_in = a.h_pad = (int)h_in, a.h_out = (int)h_out;
        a.blocks = seq_blocks(h_in, h_out, most), a.batches = seq_batches(h_in, h_out, most);
        auto end = [&](const float* g) {
            const int j = r - 1;
            ProfScope prof(KID_SEQ_VECTOR, s);
            hipLaunchKernelGGL(k_seq_finish, dim3(1), dim3(1024), 0, s, p_vec, g, Qt + (int64_t)j * h_in, sGt + (int64_t)j * h_out,
                               sigma ? sigma + j : (float*)nullptr, h_in, h_out, hdr, j, theta, eff_rank);
            DAD_LAUNCH_CHECK();
            return DAD_OK;
        };
        if (p.pair) {
            // p of a component waits for its end in its row of Qt, as the next one's first launch writes V already
            float* const vectors[2] = {panel, Ut};
            const int splits = c.tn_out.splits;
            a.slabs = splits == 1 ? Yt : part, a.nslabs = splits;
            const TnJob product = {M, static_cast<const float*>(V), splits == 1 ? Yt : part, h_in, c.tn_out.chunk, (int)h_out, splits, 1};
            for (int j = 0; j < r; ++j)
                for (int it = 0; it <= n_iter; ++it) {
                    const bool waits = it == n_iter && j + 1 < r;
                    a.j = j, a.mode = it == 0 ? SEQ_FIRST : 0, a.clear_hdr = j == 0 && it == 0;
                    a.x = G0 + (int64_t)j * h_out;
                    a.p = waits ? Qt + (int64_t)j * h_in : static_cast<float*>(V), a.h_pad = (int)(waits ? h_in : direct_npad(h_in));
                    a.p_before = j > 0 ? Qt + (int64_t)(j - 1) * h_in : nullptr;
                    a.g = vectors[it & 1], a.g_before = vectors[(it == 0 ? n_iter : it - 1) & 1];
                    DAD_TRY(seq_product<true>(a, s));
                    if (it < n_iter) DAD_TRY(direct_tn(&product, 1, 1, s, nullptr));
                }
            return end(a.g);
        }
        a.p_before = a.p, a.g_before = a.g;
        a.nslabs = a.blocks;
        for (int j = 0; j < r; ++j)
            for (int it = 0; it <= n_iter; ++it) {
                a.j = j, a.mode = (it == 0 ? SEQ_FIRST : 0) | (it == n_iter ? SEQ_LAST : 0), a.clear_hdr = j == 0 && it == 0;
                a.x = G0 + (int64_t)j * h_out;
                const int to = it & 1, from = to ^ 1;
                a.slabs = reinterpret_cast<const float*>(slabs + from * p.slab_bytes);
                a.peel = reinterpret_cast<const double*>(peels + from * p.peel_bytes);
                a.slabs_out = reinterpret_cast<float*>(slabs + to * p.slab_bytes);
                a.peel_out = reinterpret_cast<double*>(peels + to * p.peel_bytes);
                DAD_TRY(seq_product<false>(a, s));
            }
        return end(panel);
    }
    for (int j = 0; j < r; ++j) {
        {
            ProfScope prof(KID_SEQ_VECTOR, s);
            hipLaunchKernelGGL(k_seq_start, dim3(1), dim3(1024), 0, s, G0 + (int64_t)j * h_out, (const float*)sGt, j, panel,
                               h_out, hdr, j == 0 ? 1 : 0, theta, eff_rank, iters);
        }
        DAD_LAUNCH_CHECK();
        for (int it = 0; it < n_iter; ++it) {
            DAD_TRY(apply());
            {
                ProfScope prof(KID_SEQ_VECTOR, s);
                hipLaunchKernelGGL(k_seq_update, dim3(1), dim3(1024), 0, s, (const float*)Yt, (const float*)sGt, j, panel,
                                   h_out, hdr, theta, eff_rank, iters);
            }
            DAD_LAUNCH_CHECK();
        }
        DAD_TRY(last());
        {
            ProfScope prof(KID_SEQ_VECTOR, s);
            hipLaunchKernelGGL(k_seq_finish, dim3(1), dim3(1024), 0, s, p_vec, (const float*)panel,
                               Qt + (int64_t)j * h_in, sGt + (int64_t)j * h_out, sigma ? sigma + j : (float*)nullptr, h_in,
                               h_out, hdr, j, theta, eff_rank);
        }
        DAD_LAUNCH_CHECK();
    }
#undef DAD_TRY
    return DAD_OK;
}

static dad_status sequential_args_ok(const void* A, const void* D, int64_t N, int64_t h_in, int64_t h_out, dad_dtype dt,
                                     int r, int n_iter, const float* G0, const float* Qt, const float* sGt,
                                     const void* workspace) {
    if (!A || !D || !G0 || !Qt || !sGt || !workspace) return DAD_ERR_NULL;
    if (dt != DAD_F32 && dt != DAD_BF16) return DAD_ERR_DTYPE;
    if (!seq_shape_ok(N, h_in, h_out, r) || n_iter < 1) return DAD_ERR_SHAPE;
    if (!aligned16(A) || !aligned16(D) || !aligned16(G0) || !aligned16(Qt) || !aligned16(sGt) || !aligned16(workspace))
        return DAD_ERR_ALIGN;
    return DAD_OK;
}

extern "C" dad_status dad_compress_rank_sequential(const void* A, const void* D, int64_t N, int64_t h_in, int64_t h_out,
                                                   dad_dtype dt, int r, int n_iter, const float* G0, float* Qt,
                                                   float* sGt, float* sigma, void* workspace, size_t ws_bytes,
                                                   void* stream) {
    dad_status rc = sequential_args_ok(A, D, N, h_in, h_out, dt, r, n_iter, G0, Qt, sGt, workspace);
    if (rc != DAD_OK) return rc;
    const SeqPlan p = plan_sequential(N, h_in, h_out, dt);
    if (ws_bytes < p.total) return DAD_ERR_WORKSPACE;
    if ((rc = device_ready()) != DAD_OK) return rc;
    return sequential_launch(p, A, D, N, h_in, h_out, dt, r, n_iter, -1.f, G0, Qt, sGt, sigma, nullptr, nullptr, workspace,
                             (hipStream_t)stream);
}

extern "C" dad_status dad_compress_rank_adaptive(const void* A, const void* D, int64_t N, int64_t h_in, int64_t h_out,
                                                 dad_dtype dt, int r, int max_iter, float theta, const float* G0,
                                                 float* Qt, float* sGt, float* sigma, int* effective_rank,
                                                 int* iterations, void* workspace, size_t ws_bytes, void* stream) {
    dad_status rc = sequential_args_ok(A, D, N, h_in, h_out, dt, r, max_iter, G0, Qt, sGt, workspace);
    if (rc != DAD_OK) return rc;
    if (!effective_rank) return DAD_ERR_NULL;
    if (!(theta >= 0.f) || !(theta < 1.f)) return DAD_ERR_SHAPE;
    if ((reinterpret_cast<uintptr_t>(effective_rank) & 3u) || (reinterpret_cast<uintptr_t>(iterations) & 3u))
        return DAD_ERR_ALIGN;
    const SeqPlan p = plan_sequential(N, h_in, h_out, dt);
    if (ws_bytes < p.total) return DAD_ERR_WORKSPACE;
    if ((rc = device_ready()) != DAD_OK) return rc;
    return sequential_launch(p, A, D, N, h_in, h_out, dt, r, max_iter, theta, G0, Qt, sGt, sigma, effective_rank,
                             iterations, workspace, (hipStream_t)stream);
}
