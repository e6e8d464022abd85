// Orthonormalisation of the h x r iterate by Cholesky QR.  The iterate is held transposed (Yt: r x h, row j =
// column j of Y), so one round is
//   S = Y^T Y  ->  S = R^T R (upper R)  ->  G = Y R^-1,   as rows  Gt[j] = sum_i R^-1[i][j] Yt[i].
//   k_qr_gram : sums the row-chunk slabs thin_tn left of Yt on the way, forms the fp64 Gram partial of each
//               column slab on the fp64 matrix instruction, and in the workgroup that finishes last adds the
//               partials in fixed order, factorises and inverts R.
//   k_qr_apply: G = Y R^-1 with R^-1 and the sums in fp64, rounded to fp32 once.
// Products of two fp32 values are exact in fp64, so the only errors of a round are those of an fp64 Cholesky
// factorisation, G^T G - I ~ eps64 cond(Y)^2, and the final rounding.  One round is therefore the result unless
// the factor shows cond(Y) > 450 r through the upper bound ||R||_F ||R^-1||_F (or a pivot below the resolution of
// the Gram matrix): then the apply launch of the returned iterate also forms the Gram matrix of its result,
// and its last workgroup factorises again and applies the second factor to the whole panel.  That second
// round is rare (spectra steeper than fp32 contractions resolve), so it is not given launches of its own.
//
// What bounds it: latency.  Operands go straight from memory into the registers of the matrix instruction (a
// lane's four consecutive columns are four contraction steps); the serial r x r factorisation runs inside
// one wave (chol_wave.h).
#include "chol_wave.h"
#include "dad_internal.h"

namespace dad {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef f32x4 f32x4_b4 __attribute__((aligned(4)));

constexpr int QR_JOBS = 8;  // per launch
constexpr double QR_ONE_ROUND_BOUND = 2e5;  // of (||R||_F ||R^-1||_F / r)^2
// second round: the columns of a first result have unit length up to the raised pivots (at least the ratio of
// fp32 rounding noise to the floor); a column that is all but gone means that the iterate lost rank
constexpr double QR_LEAST_DIAG_2 = 1e-10;

// JT = ceil(r / 16) blocks of 16 rows; the upper block triangle of the Gram matrix has NBK blocks of 256 entries.
// A workgroup of NT threads takes COLS columns per unit (16 per wave).
template <int JT> struct QrDims {
    static constexpr int NBK = JT * (JT + 1) / 2;
    static constexpr int NR = JT == 1 ? 16 : JT == 2 ? 32 : 64;
    static constexpr int NT = JT == 1 ? 256 : 512, NW = NT / 64, COLS = 16 * NW;
    static constexpr int RB = NBK < 3 ? NBK : 3;  // blocks per round of the sum over the waves
    static constexpr int P = JT <= 2 ? 16 : 4;  // Gram partials in flight per thread
};
template <int JT> union QrShared {
    CholLds<QrDims<JT>::NR> f;
    double red[QrDims<JT>::NW][QrDims<JT>::RB][256];
    float tile[16 * JT][QrDims<JT>::COLS + 4];  // first result of one unit (second round only)
};

// Units per workgroup, a function of the iterate's own width, so that a job of a batch adds in the order of a
// call of its own.  Up to 192 columns stay in one workgroup (no partials to exchange: 3 us); partials are added by
// one workgroup, so there are at most 64 of them, and 20 of the large ones of r > 32 up to 16384 columns.
template <int JT> __host__ __device__ inline int qr_units(int64_t h) {
    constexpr int C = QrDims<JT>::COLS;
    if (h <= 192) return (int)((h + C - 1) / C);
    const int most = JT > 2 && h <= 16384 ? 20 : 64;
    return (int)((h + most * C - 1) / (most * C));
}
template <int JT> __host__ __device__ inline int qr_blocks(int64_t h) {
    const int64_t c = (int64_t)QrDims<JT>::COLS * qr_units<JT>(h);
    return (int)((h + c - 1) / c);
}

// acc[block (a, b)] += y[a] y[b]^T over 16 columns: lane (row l % 16, columns 4 (l / 16) + s)
template <int JT>
__device__ __forceinline__ void gram_add(f64x4 (&acc)[QrDims<JT>::NBK], const f32x4 (&y)[JT]) {
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        double d[JT];
#pragma unroll
        for (int a = 0; a < JT; ++a) d[a] = (double)y[a][s];
        int blk = 0;
#pragma unroll
        for (int a = 0; a < JT; ++a)
#pragma unroll
            for (int b = a; b < JT; ++b, ++blk) acc[blk] = __builtin_amdgcn_mfma_f64_16x16x4f64(d[a], d[b], acc[blk], 0, 0, 0);
    }
}

// Ends a Gram partial: the four waves are summed, the partial is published, and the workgroup that takes the
// last ticket (true) finds the symmetric total in sh.f.S.  Entry (4 v + l / 16, l % 16) of a block sits at 64 v + l.
template <int JT>
__device__ __forceinline__ bool gram_finish(QrShared<JT>& sh, const f64x4 (&acc)[QrDims<JT>::NBK], double* __restrict__ part,
                                            int nblocks, int* __restrict__ counter, int* last_s) {
    typedef QrDims<JT> D;
    constexpr int NBK = D::NBK, RB = D::RB;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int t = threadIdx.x & 255, grp = threadIdx.x >> 8;  // the second 256 threads only help to add partials
    double sum[NBK];
#pragma unroll
    for (int b0 = 0; b0 < NBK; b0 += RB) {
        __syncthreads();
#pragma unroll
        for (int b = 0; b < RB; ++b)
            if (b0 + b < NBK)
#pragma unroll
                for (int v = 0; v < 4; ++v) sh.red[wave][b][64 * v + lane] = acc[b0 + b][v];
        __syncthreads();
#pragma unroll
        for (int b = 0; b < RB; ++b)
            if (b0 + b < NBK) {
                double x = 0.0;
#pragma unroll
                for (int w = 0; w < D::NW; ++w) x += sh.red[w][b][t];
                sum[b0 + b] = x;
            }
    }
    if (nblocks > 1) {
        double* mine = part + (int64_t)blockIdx.x * NBK * 256;
        // The partials are exchanged with agent-scope accesses, which go past the caches that are not shared
        // by the XCDs: no cache has to be written back before the ticket or invalidated after it (1-2 us each).
        // The accesses are relaxed, which orders nothing by the language; on this chip a store that s_waitcnt has seen
        // arrive is visible to every later access of this scope, and the loads are issued after the ticket's value is known.
        if (grp == 0)
#pragma unroll
            for (int b = 0; b < NBK; ++b) __hip_atomic_store(mine + b * 256 + t, sum[b], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        wait_vmcnt<0>();  // this wave's stores have arrived
        __syncthreads();
        if (threadIdx.x == 0)
            *last_s = __hip_atomic_fetch_add(counter, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == nblocks - 1;
        __syncthreads();
        if (!*last_s) return false;
        if (threadIdx.x == 0) *counter = 0;
        constexpr int P = D::P, G = D::NT / 256;  // group g adds partials g, g + G, ...
#pragma unroll
        for (int b = 0; b < NBK; ++b) sum[b] = 0.0;
        for (int p0 = grp; p0 < nblocks; p0 += P * G) {
            double v[P][NBK];
#pragma unroll
            for (int u = 0; u < P; ++u)
#pragma unroll
                for (int b = 0; b < NBK; ++b) {
                    const int p = p0 + u * G < nblocks ? p0 + u * G : nblocks - 1;
                    v[u][b] = __hip_atomic_load(part + ((int64_t)p * NBK + b) * 256 + t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
#pragma unroll
            for (int u = 0; u < P; ++u)
#pragma unroll
                for (int b = 0; b < NBK; ++b) sum[b] += p0 + u * G < nblocks ? v[u][b] : 0.0;
        }
        if constexpr (G > 1) {
            double* other = &sh.red[0][0][0];
            if (grp == 1)
#pragma unroll
                for (int b = 0; b < NBK; ++b) other[b * 256 + t] = sum[b];
            __syncthreads();
#pragma unroll
            for (int b = 0; b < NBK; ++b) sum[b] += other[b * 256 + t];
        }
    }
    __syncthreads();
    if (grp == 0) {
        int blk = 0;
#pragma unroll
        for (int a = 0; a < JT; ++a)
#pragma unroll
            for (int b = a; b < JT; ++b, ++blk) {
                const int i = 16 * a + 4 * wave + (lane >> 4), j = 16 * b + (lane & 15);
                sh.f.S[i][j] = sum[blk];
                if (a != b) sh.f.S[j][i] = sum[blk];
            }
    }
    __syncthreads();
    return true;
}

// Pivot ranges of the two factors of a job.
__device__ __forceinline__ double* qr_range(const QrJob& jb) { return reinterpret_cast<double*>(reinterpret_cast<char*>(jb.hdr) + 128); }

template <int JT, int CAP>
__global__ __launch_bounds__(QrDims<JT>::NT) void k_qr_gram(JobTable<QrJob, CAP> tb, int r) {
    __shared__ QrShared<JT> sh;
    __shared__ int last_s;
    const QrJob& jb = tb.j[blockIdx.y];
    const int64_t h = jb.h;
    const int nblocks = qr_blocks<JT>(h);
    if ((int)blockIdx.x >= nblocks) return;
    const float* __restrict__ Y = jb.Y;
    float* __restrict__ Ysum = jb.Ysum;
    const int splits = jb.splits;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, i = lane & 15, q = lane >> 4;
    f64x4 acc[QrDims<JT>::NBK];
#pragma unroll
    for (int b = 0; b < QrDims<JT>::NBK; ++b) acc[b] = f64x4{0.0, 0.0, 0.0, 0.0};
    const int64_t slab = (int64_t)r * h;
    const int units = qr_units<JT>(h);
    for (int u = 0; u < units; ++u) {
        const int64_t c0 = ((int64_t)blockIdx.x * units + u) * QrDims<JT>::COLS + wave * 16;
        if (c0 >= h) break;
        const int64_t c = c0 + 4 * q;
        f32x4 y[JT];
        if (h < 4) {  // narrower than one load
#pragma unroll
            for (int a = 0; a < JT; ++a)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    y[a][e] = 0.f;
                    if (16 * a + i < r && c + e < h) {
                        const int64_t at = (int64_t)(16 * a + i) * h + c + e;
                        for (int s = 0; s < splits; ++s) y[a][e] += Y[s * slab + at];
                        if (Ysum) Ysum[at] = y[a][e];
                    }
                }
        } else {
            const int64_t cc = c < h - 4 ? c : h - 4;  // the last columns: loaded from h - 4 on, those of the lane before masked
            // all JT rows of eight slabs in flight at a time (the sum is latency bound), added in slab order
            const float* src[JT];
#pragma unroll
            for (int a = 0; a < JT; ++a) {
                src[a] = Y + (int64_t)(16 * a + i < r ? 16 * a + i : r - 1) * h + cc;
                y[a] = *reinterpret_cast<const f32x4_b4*>(src[a]);
            }
            for (int s = 1; s < splits; s += 8) {
                f32x4 v[8][JT];
#pragma unroll
                for (int e = 0; e < 8; ++e)
#pragma unroll
                    for (int a = 0; a < JT; ++a)
                        v[e][a] = *reinterpret_cast<const f32x4_b4*>(src[a] + (s + e < splits ? s + e : splits - 1) * slab);
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if (s + e < splits)
#pragma unroll
                        for (int a = 0; a < JT; ++a) y[a] += v[e][a];
            }
#pragma unroll
            for (int a = 0; a < JT; ++a) {
                const bool in = 16 * a + i < r && c < h;
                if (Ysum && in) *reinterpret_cast<f32x4_b4*>(Ysum + (int64_t)(16 * a + i) * h + cc) = y[a];
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (!in || cc + e < c) y[a][e] = 0.f;
            }
        }
        gram_add<JT>(acc, y);
    }
    if (!gram_finish<JT>(sh, acc, jb.part, nblocks, jb.hdr + 16, &last_s)) return;
    chol_factor<QrDims<JT>::NR>(sh.f, r, 0.0, jb.rinv, jb.flag, qr_range(jb));
}

// One wave: 16 columns from c0 of Gt = R^-T Yt.  out[b][v]: row 16 b + 4 v + lane / 16, column c0 + lane % 16.
template <int JT>
__device__ __forceinline__ void apply_columns(const double (&ri)[QrDims<JT>::NBK][4], const float* Yt, int64_t h, int r,
                                              int64_t c0, f64x4 (&out)[JT]) {
    const int lane = threadIdx.x & 63, li = lane & 15, q = lane >> 4;
    const int64_t c = c0 + li < h ? c0 + li : h - 1;
    float y[JT][4];
#pragma unroll
    for (int a = 0; a < JT; ++a)
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const int row = 16 * a + 4 * s + q;
            y[a][s] = Yt[(int64_t)(row < r ? row : r - 1) * h + c];  // rows >= r meet zeros of R^-1
        }
    int blk = 0;
#pragma unroll
    for (int b = 0; b < JT; ++b) {
        out[b] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int a = 0; a <= b; ++a, ++blk)
#pragma unroll
            for (int s = 0; s < 4; ++s) out[b] = __builtin_amdgcn_mfma_f64_16x16x4f64(ri[blk][s], (double)y[a][s], out[b], 0, 0, 0);
    }
}

// The lane's entries of R^-1 (block column b of output rows, block row a <= b): row operand of the products above.
template <int JT>
__device__ __forceinline__ void load_rinv(double (&ri)[QrDims<JT>::NBK][4], const double* rinv, int r) {
    const int lane = threadIdx.x & 63, li = lane & 15, q = lane >> 4;
    int blk = 0;
#pragma unroll
    for (int b = 0; b < JT; ++b)
#pragma unroll
        for (int a = 0; a <= b; ++a, ++blk)
#pragma unroll
            for (int s = 0; s < 4; ++s) {
                const int i = 16 * a + 4 * s + q, j = 16 * b + li;
                const bool in = i <= j && j < r;
                const double v = rinv[in ? i * r + j : 0];
                ri[blk][s] = in ? v : 0.0;
            }
}

// Gt <- R^-T Yt (Gt may be Yt: a workgroup reads its columns before it writes them), with an optional bf16 copy
// (the panel of the next thin_nn).  FINAL: the returned iterate, with the second round where the first
// factor asks for it (see the head of this file).
template <int JT, bool FINAL, int CAP>
__global__ __launch_bounds__(FINAL ? QrDims<JT>::NT : 256) void k_qr_apply(JobTable<QrJob, CAP> tb, int r) {
    const QrJob& jb = tb.j[blockIdx.y];
    const int64_t h = jb.h;
    constexpr int COLS = FINAL ? QrDims<JT>::COLS : 64;  // of a workgroup
    if ((int64_t)blockIdx.x * COLS >= h) return;
    const float* Yt = jb.Ysum ? jb.Ysum : jb.Y;
    float* Gt = jb.Gt;
    bf16_t* gt_bf16 = jb.gt_bf16;
    double* rinv = jb.rinv;
    double* rinv2 = rinv + DAD_MAX_RANK * DAD_MAX_RANK;
    double* range = qr_range(jb);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, li = lane & 15, q = lane >> 4;
    double ri[QrDims<JT>::NBK][4];
    load_rinv<JT>(ri, rinv, r);
    auto write = [&](const f64x4 (&g)[JT], int64_t c, bool with_bf16) {
        if (c >= h) return;
#pragma unroll
        for (int b = 0; b < JT; ++b)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int row = 16 * b + 4 * v + q;
                if (row < r) {
                    const float x = (float)g[b][v];
                    Gt[(int64_t)row * h + c] = x;
                    if (with_bf16) gt_bf16[(int64_t)row * h + c] = f32_to_bf16(x);
                }
            }
    };
    if constexpr (!FINAL) {
        const int64_t c0 = (int64_t)blockIdx.x * 64 + wave * 16;
        f64x4 g[JT];
        apply_columns<JT>(ri, Yt, h, r, c0, g);
        write(g, c0 + li, gt_bf16 != nullptr);
    } else {
        __shared__ QrShared<JT> sh;
        __shared__ int last_s;
        const bool again = range[0] > 0.0 && !(range[1] <= QR_ONE_ROUND_BOUND);  // uniform over the grid
        if (!again) {
            const int64_t c0 = (int64_t)blockIdx.x * COLS + wave * 16;
            f64x4 g[JT];
            apply_columns<JT>(ri, Yt, h, r, c0, g);
            write(g, c0 + li, gt_bf16 != nullptr);
            return;
        }
        // the second round: few workgroups, as one of them adds their Gram partials
        const int nblocks = qr_blocks<JT>(h);
        if ((int)blockIdx.x >= nblocks) return;
        f64x4 acc[QrDims<JT>::NBK];
#pragma unroll
        for (int b = 0; b < QrDims<JT>::NBK; ++b) acc[b] = f64x4{0.0, 0.0, 0.0, 0.0};
        const int units = qr_units<JT>(h);
        for (int u = 0; u < units; ++u) {
            const int64_t cu = ((int64_t)blockIdx.x * units + u) * QrDims<JT>::COLS, c = cu + wave * 16 + li;
            if (cu >= h) break;
            f64x4 g[JT];
            apply_columns<JT>(ri, Yt, h, r, cu + wave * 16, g);
            write(g, c, false);
            if (u) __syncthreads();
#pragma unroll
            for (int b = 0; b < JT; ++b)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int row = 16 * b + 4 * v + q;
                    sh.tile[row][wave * 16 + li] = row < r && c < h ? (float)g[b][v] : 0.f;
                }
            __syncthreads();
            f32x4 y[JT];
#pragma unroll
            for (int a = 0; a < JT; ++a) y[a] = *reinterpret_cast<const f32x4*>(&sh.tile[16 * a + li][wave * 16 + 4 * q]);
            gram_add<JT>(acc, y);
        }
        __syncthreads();
        __threadfence();  // the first result leaves before the ticket
        if (!gram_finish<JT>(sh, acc, jb.part, nblocks, jb.hdr + 16, &last_s)) return;
        __threadfence();
        chol_factor<QrDims<JT>::NR>(sh.f, r, QR_LEAST_DIAG_2, rinv2, jb.flag, range + 2);
        __threadfence();
        __syncthreads();
        load_rinv<JT>(ri, rinv2, r);
        for (int64_t c0 = wave * 16; c0 < h; c0 += QrDims<JT>::COLS) {
            f64x4 g[JT];
            apply_columns<JT>(ri, Gt, h, r, c0, g);
            write(g, c0 + li, gt_bf16 != nullptr);
        }
    }
}

template <int JT> static size_t part_bytes(int64_t h) {
    const int64_t whole = ceil_div(h, QrDims<JT>::COLS);
    const int nb = whole < 64 ? (int)whole : 64;  // at least the blocks of any iterate up to h wide
    return (size_t)nb * QrDims<JT>::NBK * 256 * sizeof(double);
}

// Bytes of Gram partials of any iterate up to h wide.
size_t qr_part_bytes(int64_t h, int r) {
    return r <= 16 ? part_bytes<1>(h) : r <= 32 ? part_bytes<2>(h) : r <= 48 ? part_bytes<3>(h) : part_bytes<4>(h);
}

template <int JT>
static dad_status qr(const QrJob* jobs, int count, int r, bool final, hipStream_t s) {
    int nb = 0;
    int64_t h = 0;
    for (int i = 0; i < count; ++i) {
        if (qr_blocks<JT>(jobs[i].h) > nb) nb = qr_blocks<JT>(jobs[i].h);
        if (jobs[i].h > h) h = jobs[i].h;
    }
    constexpr int NT = QrDims<JT>::NT;
    const dim3 grid((unsigned)nb, (unsigned)count), cols((unsigned)ceil_div(h, QrDims<JT>::COLS), (unsigned)count);
    {
        ProfScope prof(KID_GRAM, s);
        launch_jobs<QR_JOBS>(jobs, count, [&](auto tb, auto cap) {
            hipLaunchKernelGGL((k_qr_gram<JT, decltype(cap)::value>), grid, dim3(NT), 0, s, tb, r);
        });
    }
    DAD_LAUNCH_CHECK();
    if (final) {
        ProfScope prof(KID_APPLY, s);
        launch_jobs<QR_JOBS>(jobs, count, [&](auto tb, auto cap) {
            hipLaunchKernelGGL((k_qr_apply<JT, true, decltype(cap)::value>), cols, dim3(NT), 0, s, tb, r);
        });
    } else {
        ProfScope prof(KID_APPLY2, s);
        launch_jobs<QR_JOBS>(jobs, count, [&](auto tb, auto cap) {
            hipLaunchKernelGGL((k_qr_apply<JT, false, decltype(cap)::value>), dim3((unsigned)ceil_div(h, 64), (unsigned)count), dim3(256), 0, s, tb, r);
        });
    }
    DAD_LAUNCH_CHECK();
    return DAD_OK;
}

dad_status launch_cholqr(const QrJob* jobs, int count, int r, bool final, hipStream_t s) {
    for (int i = 0; i < count; i += QR_JOBS) {
        const int n = count - i < QR_JOBS ? count - i : QR_JOBS;
        const dad_status rc = r <= 16   ? qr<1>(jobs + i, n, r, final, s)
                              : r <= 32 ? qr<2>(jobs + i, n, r, final, s)
                              : r <= 48 ? qr<3>(jobs + i, n, r, final, s)
                                        : qr<4>(jobs + i, n, r, final, s);
        if (rc != DAD_OK) return rc;
    }
    return DAD_OK;
}

}  // namespace dad
