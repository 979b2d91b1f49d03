// Products of steps 4-5 of Algorithm 1 (Eq. 8) on the fp32 matrix cores:
//
//   U = V^T K(X_r, X_t)      (k x m)      or   G = K(X_r, X_t) R   (s x l)
//   W = D (U R)              (k x l)           W = D (V^T G)       (k x l)
//   alpha_r += c V W                           (same)
//
// with V the s x k eigenvector block, D its diagonal scale, R the batch
// residual and K(X_r, X_t) the subsample columns kept by step 2. All are
// thin products (one side of at most a few hundred) whose depth may be long
// (s = 20000), so one kernel serves them all:
//
//   C[p] = sum over depth chunk p of A(i, kk) B(kk, j)
//
// with B row-major (depth x N) and A either row-major (M x depth) or the
// transpose of a row-major (depth x M) matrix. A workgroup of 4 waves owns
// a 64 x 64 output tile, each wave a 32 x 32 block on
// v_mfma_f32_32x32x2f32; operands are staged through LDS in 32-deep stages
// (depth-major, so a lane's operand read is one conflict-free LDS word),
// two stages deep: the next stage is fetched while the current one feeds
// the MFMAs.
// Depth is split into chunks (`kc`, one partial slice each, summed by the
// reduction kernels in slice order) so that enough workgroups exist, and
// inside a chunk the accumulation is blocked: the MFMA accumulator is
// restarted every 64 depth and added into a running sum, so no float32
// chain is longer than 32 MFMA steps plus one addition per block. (The
// component of these products along the top eigenvector sums terms that
// largely cancel; a single chain over the whole depth visibly raised the
// prediction error.)
//
// The last product's epilogue adds coef * (V W)[i, j] straight into
// alpha[r[i], j] (the rows r are distinct, so no two lanes write one
// element).
#include "ep_device.h"
#include "ep_internal.h"
#include "split.h"

namespace ep {

namespace {

constexpr int kTM = 64, kTN = 64;     // output tile
constexpr int kKS = 32;               // depth per LDS stage
constexpr int kBlk = 64;              // depth per accumulation block
constexpr int kGThreads = 256;
constexpr int kPadA = 4, kPadB = 4;   // LDS row padding (floats)

// The first `len` (of four) floats at `at`, zero after them; nothing at `at`
// is read when len <= 0 (the load then goes to `safe`). No branch: a load
// inside one is waited for where the paths join, and the four loads of a
// stage would each cost their latency.
__device__ __forceinline__ float4 ld4(const float* at, int64_t len, const float* safe) {
    float4 v = *reinterpret_cast<const float4*>(len > 0 ? at : safe);
    v.x = len > 0 ? v.x : 0.f;
    v.y = len > 1 ? v.y : 0.f;
    v.z = len > 2 ? v.z : 0.f;
    v.w = len > 3 ? v.w : 0.f;
    return v;
}

template <bool A_T, bool SCATTER>
__global__ void __launch_bounds__(kGThreads) thin_gemm_kernel(ThinGemmArgs p) {
    // two LDS stages: the next stage's operands are fetched into registers
    // while the MFMAs read the current one, so one barrier per stage
    __shared__ float As[2][kKS][kTM + kPadA];
    __shared__ float Bs[2][kKS][kTN + kPadB];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int tm = (int)((p.M + kTM - 1) / kTM);
    const int tn = (int)((p.N + kTN - 1) / kTN);
    const int tile = (int)(blockIdx.x % (unsigned)(tm * tn));
    const int chunk = (int)(blockIdx.x / (unsigned)(tm * tn));
    const int64_t i0 = (int64_t)(tile / tn) * kTM;
    const int64_t j0 = (int64_t)(tile % tn) * kTN;
    const int64_t k_lo = (int64_t)chunk * p.kc;
    const int64_t k_hi = min(p.K, k_lo + p.kc);
    const int wm = wave & 1, wn = wave >> 1;

    floatx16 acc, sum;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        acc[v] = 0.f;
        sum[v] = 0.f;
    }
    // this thread's share of a stage: two quads of A, two of B
    float4 ra[2], rb[2];
    auto fetch = [&](int64_t k0) {
        const int64_t kd = min((int64_t)kKS, k_hi - k0);   // valid depth of the stage
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const int q = tid + e * kGThreads;
            if (A_T) {
                // A(i, kk) = A[kk * lda + i]: quad of (depth, 4 rows)
                const int kk = q / (kTM / 4), ii = 4 * (q % (kTM / 4));
                ra[e] = ld4(p.A + (k0 + kk) * p.lda + i0 + ii, kk < kd ? p.M - i0 - ii : 0, p.A);
            } else {
                // A(i, kk) = A[i * lda + kk]: quad of (row, 4 depth)
                const int ii = q / (kKS / 4), kk = 4 * (q % (kKS / 4));
                ra[e] = ld4(p.A + (i0 + ii) * p.lda + k0 + kk, i0 + ii < p.M ? kd - kk : 0, p.A);
            }
            const int kk = q / (kTN / 4), jj = 4 * (q % (kTN / 4));
            rb[e] = ld4(p.B + (k0 + kk) * p.ldb + j0 + jj, kk < kd ? p.N - j0 - jj : 0, p.B);
        }
    };
    // A tile -> As[depth][row], B tile -> Bs[depth][col]
    auto stash = [&](int buf) {
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            const int q = tid + e * kGThreads;
            if (A_T) {
                const int kk = q / (kTM / 4), ii = 4 * (q % (kTM / 4));
                *reinterpret_cast<float4*>(&As[buf][kk][ii]) = ra[e];
            } else {
                const int ii = q / (kKS / 4), kk = 4 * (q % (kKS / 4));
                As[buf][kk][ii] = ra[e].x;
                As[buf][kk + 1][ii] = ra[e].y;
                As[buf][kk + 2][ii] = ra[e].z;
                As[buf][kk + 3][ii] = ra[e].w;
            }
            const int kk = q / (kTN / 4), jj = 4 * (q % (kTN / 4));
            *reinterpret_cast<float4*>(&Bs[buf][kk][jj]) = rb[e];
        }
    };
    int in_block = 0;
    int buf = 0;
    if (k_lo < k_hi) fetch(k_lo);
    for (int64_t k0 = k_lo; k0 < k_hi; k0 += kKS, buf ^= 1) {
        // the stage written here was last read two stages ago, before the
        // previous barrier
        stash(buf);
        __syncthreads();
        if (k0 + kKS < k_hi) fetch(k0 + kKS);
        const int h = lane >> 5, r = lane & 31;
#pragma unroll
        for (int s2 = 0; s2 < kKS / 2; ++s2) {
            const float a = As[buf][2 * s2 + h][wm * 32 + r];
            const float b = Bs[buf][2 * s2 + h][wn * 32 + r];
            acc = mfma(a, b, acc);
        }
        in_block += kKS;
        if (in_block == kBlk || k0 + kKS >= k_hi) {
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                sum[v] += acc[v];
                acc[v] = 0.f;
            }
            in_block = 0;
        }
    }

    // element v of this lane: row acc_row(v, lane), column lane % 32
    const int64_t col = j0 + wn * 32 + (lane & 31);
    if (SCATTER) {
        if (col >= p.N_valid) return;
        // all rows and old values first: a store between two loads would
        // order them, and each update would cost its own round trip
        int64_t r[16];
        float old[16];
#pragma unroll
        for (int v = 0; v < 16; ++v)
            r[v] = p.r[min(i0 + wm * 32 + acc_row(v, lane), p.M - 1)];
#pragma unroll
        for (int v = 0; v < 16; ++v) old[v] = p.alpha[r[v] * p.ldalpha + col];
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            if (i0 + wm * 32 + acc_row(v, lane) < p.M) {
                const float a = old[v] + p.coef * sum[v];
                p.alpha[r[v] * p.ldalpha + col] = a;
                if (p.planes) store_weight(p.planes, weight_elem(r[v], col, p.lt), a);
            }
        }
    } else {
        if (col >= p.N) return;
        float* C = p.C + (int64_t)chunk * p.slice;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int64_t row = i0 + wm * 32 + acc_row(v, lane);
            if (row < p.M) C[row * p.ldc + col] = sum[v];
        }
    }
}

// out[i, j] = scale_i * sum_p part[p][i, j] (scale = 1 without Dk), slices
// summed in order.
template <class T>
__global__ void __launch_bounds__(256) sum_slices_kernel(const float* part, int slices,
                                                         int64_t slice, int64_t rows, int64_t cols,
                                                         int64_t ld, const float* Dk, float* out,
                                                         int64_t ldo) {
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= rows * cols) return;
    const int64_t i = e / cols, j = e - i * cols;
    const float* at = part + i * ld + j;
    T f = 0;
    int s = 0;
    for (; s + 8 <= slices; s += 8) {           // eight loads in flight
        float v[8];
#pragma unroll
        for (int x = 0; x < 8; ++x) v[x] = at[(int64_t)(s + x) * slice];
#pragma unroll
        for (int x = 0; x < 8; ++x) f += v[x];
    }
    for (; s < slices; ++s) f += at[(int64_t)s * slice];
    out[i * ldo + j] = (float)(Dk ? Dk[i] * f : f);
}

}  // namespace

ThinGemmPlan thin_gemm_plan(int64_t M, int64_t N, int64_t K, int min_groups, int64_t min_depth) {
    ThinGemmPlan pl;
    const int64_t tiles = ceil_div(M, kTM) * ceil_div(N, kTN);
    // depth chunks: enough workgroups to fill the chip, chunks of whole
    // accumulation blocks and at least min_depth deep. A stage of 32 costs a
    // workgroup about 1.6 us however few of them run, so short products want
    // chunks of one block (20 x 256 x 500: 26 us in one chunk, 7 in eight).
    int64_t chunks = std::max<int64_t>(1, ceil_div(min_groups, tiles));
    chunks = std::min<int64_t>(chunks, std::max<int64_t>(1, K / min_depth));
    chunks = std::min<int64_t>(chunks, 64);
    pl.kc = round_up(ceil_div(K, chunks), kBlk);
    pl.chunks = (int)ceil_div(K, pl.kc);
    pl.tiles = tiles;
    return pl;
}

hipError_t thin_gemm_launch(const ThinGemmArgs& a, const ThinGemmPlan& pl, bool a_t, bool scatter,
                            hipStream_t st) {
    if (a.M <= 0 || a.N <= 0) return hipSuccess;
    if ((a.lda & 3) || (a.ldb & 3) || (reinterpret_cast<uintptr_t>(a.A) & 15) ||
        (reinterpret_cast<uintptr_t>(a.B) & 15))
        return hipErrorInvalidValue;
    if (scatter && pl.chunks != 1) return hipErrorInvalidValue;
    ThinGemmArgs b = a;
    b.kc = pl.kc;
    const dim3 grid((unsigned)(pl.tiles * pl.chunks));
    if (a_t) {
        if (scatter) hipLaunchKernelGGL((thin_gemm_kernel<true, true>), grid, dim3(kGThreads), 0, st, b);
        else hipLaunchKernelGGL((thin_gemm_kernel<true, false>), grid, dim3(kGThreads), 0, st, b);
    } else {
        if (scatter) hipLaunchKernelGGL((thin_gemm_kernel<false, true>), grid, dim3(kGThreads), 0, st, b);
        else hipLaunchKernelGGL((thin_gemm_kernel<false, false>), grid, dim3(kGThreads), 0, st, b);
    }
    return hipGetLastError();
}

hipError_t launch_sum_slices(const float* part, int slices, int64_t slice, int64_t rows,
                             int64_t cols, int64_t ld, const float* Dk, float* out, int64_t ldo,
                             bool f64, hipStream_t st) {
    if (rows <= 0 || cols <= 0) return hipSuccess;
    const int64_t count = rows * cols;
    hipLaunchKernelGGL(f64 ? sum_slices_kernel<double> : sum_slices_kernel<float>,
                       dim3((unsigned)ceil_div(count, 256)), dim3(256), 0, st, part, slices, slice,
                       rows, cols, ld, Dk, out, ldo);
    return hipGetLastError();
}

}  // namespace ep
