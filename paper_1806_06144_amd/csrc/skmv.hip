// Fused kernel-block contraction on the 16-bit matrix cores of gfx950:
//
//   out[q, :] = sum_j k(q, c_j) W[j, :]      (Algorithm 1 step 2, prediction)
//
// the same pass as kmv.hip, with both float32 products replaced by sums of
// 16-bit products (split.h says what these keep): distances as three fp16
// products of two planes, four where rows need it, the contraction with the
// weights as six bf16 products of three planes, all accumulated in float32.
// The fp16 / bf16 MFMA runs 16 times as many products per cycle as the fp32
// one, so the distance product costs 3/16 and the contraction 6/16 of what it
// did.
//
// The matrix pipes are busy 44 to 65 % of the cycles, at 2.4 GHz in a short
// step and 1.7 to 2.05 GHz, under the card's power limit, in longer ones; the
// rest are waits inside the workgroups. Counting three and six products: 1.0
// PFLOP/s at 60000 x 784, 10 labels, 1310 queries (382 us; the float32 pass
// 1070 us), 1.42 with 10000 queries, 0.92 at 1.1 M x 440, 144 labels, 1257
// queries (6.55 ms; float32 12.9 ms); a large library product reaches 1.2.
//
// Four waves share a panel of 128 centres through LDS (direct-to-LDS loads
// of 32 features, three stages ahead in four slots, one barrier per stage);
// each wave owns 64 queries (32 beyond 16 labels), whose operands it reads
// from the L2 one stage ahead. Kernel values never leave the registers: the
// accumulators of the distance product are the operands of the contraction
// (weight_elem in split.h orders the weights to match). Two workgroups fit a
// CU, so one's epilogue runs beside the other's products; a version with
// twice the queries per wave and one workgroup per CU took 7.8 ms instead of
// 6.6 at 144 labels.
#include "ep_device.h"
#include "ep_internal.h"
#include "launch.h"
#include "split.h"

#include <algorithm>
#include <cstdlib>
#include <type_traits>

namespace ep {

namespace {

constexpr int kSThreads = 256;                       // 4 waves
constexpr int kSlotQuads = kCPanel / 16 * 2 * 64;    // 16-byte quads of one 32-feature stage

// ---- packing ---------------------------------------------------------------

// Packs 16 rows per workgroup: row maxima first unless the scales are given,
// then the two scaled fp16 planes, and from them the norms of the packed rows
// (float64 sums of (hi + lo)^2). Rows past `rows` and gathered rows out of
// [0, n) are zero (norm 0, scale 1).
template <bool VEC>
__global__ void __launch_bounds__(1024) pack_rows_kernel(PackArgs p) {
    __shared__ float s_inv[16];
    __shared__ int64_t s_row[16];
    __shared__ double s_sum[16][2][16];              // [wave][(hi + lo)^2, lo^2][row]
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, waves = blockDim.x >> 6;
    const int64_t tiles = (p.rows + p.P - 1) / p.P * (p.P / 16);
    for (int64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        if (tid < 16) {
            const int64_t b = tile * 16 + tid;
            int64_t src = b < p.rows ? b : -1;
            if (p.idx && src >= 0) {
                src = p.idx[b];
                if (src < 0 || src >= p.n) {
                    atomicOr(p.err, 1);
                    src = -1;
                }
            }
            s_row[tid] = src;
            if (p.inv_in) s_inv[tid] = src >= 0 ? p.inv_in[src] : 1.f;
        }
        __syncthreads();
        if (!p.inv_in) {
            for (int r = wave; r < 16; r += waves) {
                const int64_t src = s_row[r];
                float mx = 0.f;
                if (src >= 0) {
                    const float* x = p.X + src * p.d;
                    for (int64_t j = lane; j < p.d; j += 512) {
                        float v[8];                  // (eight loads in flight; repeats of the last)
#pragma unroll
                        for (int e = 0; e < 8; ++e) v[e] = x[min(j + 64 * e, p.d - 1)];
#pragma unroll
                        for (int e = 0; e < 8; ++e) mx = fmaxf(mx, fabsf(v[e]));
                    }
                }
                for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_down(mx, off, 64));
                if (lane == 0) {
                    // largest element into [2^14, 2^15); exponents below -49
                    // share one scale, so that the product of two inverse
                    // scales stays a normal float32 (2^-63, whose square is
                    // the smallest normal one, still has 24 bits in lo)
                    const int e =
                        mx == 0.f ? 14 : max(-49, (int)(__builtin_bit_cast(unsigned, mx) >> 23) - 127);
                    s_inv[r] = mx == __builtin_inff()
                                   ? mx
                                   : __builtin_bit_cast(float, (unsigned)(e - 14 + 127) << 23);
                }
            }
            __syncthreads();
        }
        const int row = lane & 15, g = lane >> 4;
        const int64_t src = s_row[row];
        const float sc = 1.f / s_inv[row];     // (a power of two: exact; zero for an infinite row)
        const float* x = p.X + (src >= 0 ? src : 0) * p.d;
        const int64_t t_panel = p.P / 16;
        char* out = p.out + (tile / t_panel) * p.panel + (tile % t_panel) * 2 * kFragBytes + lane * 16;
        double sum = 0.0, sum_lo = 0.0;
        for (int64_t ks = wave; ks < p.nk; ks += waves) {
            const int64_t c0 = ks * 32 + 8 * g;
            const float flip = ks >= p.neg0 && ks < p.neg1 ? -1.f : 1.f;
            float v[8];
            if (VEC) {
                const float4 z = make_float4(0.f, 0.f, 0.f, 0.f);
                const float4 a = src >= 0 && c0 < p.d ? *reinterpret_cast<const float4*>(x + c0) : z;
                const float4 b =
                    src >= 0 && c0 + 4 < p.d ? *reinterpret_cast<const float4*>(x + c0 + 4) : z;
                v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
                v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
            } else {
#pragma unroll
                for (int j = 0; j < 8; ++j) v[j] = src >= 0 && c0 + j < p.d ? x[c0 + j] : 0.f;
            }
            half8 hi, lo;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                float s = v[j] * sc * flip;
                if (!__builtin_isfinite(v[j])) {
                    s = __builtin_isinf(v[j]) ? __builtin_copysignf(flip, v[j] * flip) : 0.f;
                    if (v[j] != v[j]) sum += v[j];
                }
                const _Float16 h = (_Float16)s;
                hi[j] = h;
                lo[j] = (_Float16)(s - (float)h);
                const double ql = (double)(float)lo[j], q = (double)(float)h + ql;
                sum += q * q;
                if (p.lolo) sum_lo += ql * ql;
            }
            char* o = out + ks * t_panel * 2 * kFragBytes;
            *reinterpret_cast<half8*>(o) = hi;
            *reinterpret_cast<half8*>(o + kFragBytes) = lo;
        }
        for (int off = 32; off >= 16; off >>= 1) {
            sum += __shfl_down(sum, off, 64);
            sum_lo += __shfl_down(sum_lo, off, 64);
        }
        if (lane < 16) {
            s_sum[wave][0][lane] = sum;
            s_sum[wave][1][lane] = sum_lo;
        }
        __syncthreads();
        if (wave == 0) {
            double sq = 0.0, sl = 0.0;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int w = 4 * e + g;
                if (w < waves) {
                    sq += s_sum[w][0][row];
                    sl += s_sum[w][1][row];
                }
            }
            for (int off = 32; off >= 16; off >>= 1) {
                sq += __shfl_down(sq, off, 64);
                sl += __shfl_down(sl, off, 64);
            }
            if (lane < 16) {
                const float inv = s_inv[lane];
                const int64_t b = tile * 16 + lane;
                const int64_t panel = b / p.P, at = b % p.P;
                float* meta = reinterpret_cast<float*>(p.out + panel * p.panel +
                                                       p.nk * (p.P / 16) * 2 * kFragBytes);
                meta[at] = (float)(sq * inv * inv);
                meta[p.P + at] = inv;
                if (p.inv_out && b < p.rows) p.inv_out[b] = inv;
                // (the same value from every row that needs it)
                if (p.lolo && sl > kLoLoMax * sq) p.lolo[panel] = 1;
            }
        }
        __syncthreads();               // the next tile overwrites rows, scales, sums
    }
}

// Planes of a whole weight matrix (rows x l floats, leading dimension ldw),
// labels up to lt tiles and rows up to whole groups of 32 zero. A thread packs
// the eight weights of a lane of an operand (weight_elem), so that stores are
// 16 bytes beside each other: 1.28 M x 1000 in 2.6 ms (5.1 GB in, 7.7 out, 4.9
// TB/s); one thread a weight, 2-byte stores 16 bytes apart, took 12.5.
__global__ void __launch_bounds__(256) pack_weights_kernel(const float* W, int64_t rows, int64_t l,
                                                           int64_t ldw, int64_t lt,
                                                           unsigned short* planes) {
    typedef unsigned short ushortx8 __attribute__((ext_vector_type(8)));
    const int64_t lanes = (rows + 31) / 32 * lt * 64;
    for (int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x; e < lanes;
         e += (int64_t)gridDim.x * 256) {
        const int lane = (int)(e & 63);
        const int64_t frag = e >> 6, group = frag / lt;
        const int64_t j = 16 * (frag - group * lt) + (lane & 15);
        const int64_t c0 = 32 * group + 4 * (lane >> 4);
        ushortx8 h, m, o;
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int64_t c = c0 + 16 * (i >> 2) + (i & 3);
            unsigned short a, b, d;
            split_weight(c < rows && j < l ? W[c * ldw + j] : 0.f, a, b, d);
            h[i] = a;
            m[i] = b;
            o[i] = d;
        }
        ushortx8* at = reinterpret_cast<ushortx8*>(planes) + frag * 3 * 64 + lane;
        at[0] = h;
        at[64] = m;
        at[128] = o;
    }
}

// ---- the fused pass --------------------------------------------------------

// One workgroup = 4 waves owns a contiguous range of centre panels of 128
// rows, walked panel by panel, for a tile of queries: the waves form 8 / CW
// groups of CW blocks of 16 centres by CW / 2 groups of QB blocks of 16
// queries. CW = 8 gives every wave all centres of the panel and queries of
// its own (64 QB in all); CW = 2 gives the waves a quarter of the panel each
// and the same 16 QB queries, for calls of few rows, where otherwise three
// waves of four would idle: one row against 60000 x 784 80 -> 35 us (the
// packed centres at 5.4 TB/s), 48 rows against 1.1 M x 440 with 144 labels
// 1130 -> 595 us (centres and weights at 4.9 TB/s: both at the rate of a
// large copy). For many queries CW = 4 is slower than CW = 8: it moves the
// same centres for half the queries (10000 rows against 60000 x 784, 2.68
// against 2.11 ms).
// LT = 0: the kernel values themselves are the result, written as the operand
// planes of wmul_kernel (16 queries x 32 centres, three bf16 planes; those of
// odd 32-centre groups negated).
// LL: some panels of centres need the products of the low planes (split.h).
// The branch alone costs 5 to 8 % where the accumulators fill the registers
// (10 labels, 60000 x 784: 1310 queries 456 -> 479 us, 10000 queries 2044 ->
// 2207 us), so problems without such a panel run without it. With the
// products in every panel (the same centres with a constant column of 64.03):
// 398 -> 483 us and 2.44 -> 2.98 ms a pass.
template <int KIND, int LT, int QB, int CW, bool LL>
__global__ void __launch_bounds__(kSThreads, 2) skmv_kernel(SplitArgs p) {
    static_assert(CW == 8 || LT > 0, "stored kernel values: CW = 8");
    constexpr int kWQ = 16 * QB;                     // queries per wave
    constexpr int kSQ = CW / 2 * kWQ;
    constexpr int kCG = 8 / CW;                      // centre groups
    __shared__ uintx4 xs0[kSlotQuads];
    __shared__ uintx4 xs1[kSlotQuads];
    __shared__ uintx4 xs2[kSlotQuads];
    __shared__ uintx4 xs3[kSlotQuads];
    __shared__ __attribute__((aligned(16))) float s_meta[2 * kCPanel];   // norms, inverse scales

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 15, g = lane >> 4;
    const int tq = (int)((p.nq + kSQ - 1) / kSQ);
    const int split = (int)blockIdx.x / tq;
    const int qtile = (int)blockIdx.x - split * tq;
    const int ntile = (int)((p.nc + kCPanel - 1) / kCPanel);
    const int t0 = (int)min((int64_t)ntile, split * p.tps);
    const int t1 = (int)min((int64_t)ntile, t0 + p.tps);
    const int nk = (int)p.nk;

    // this wave's queries, inside one packed panel (a wave past the last
    // query only helps to move the centres)
    const int wq = wave / kCG, wc = wave % kCG;
    [[maybe_unused]] const float sgn = wc & 1 ? -1.f : 1.f;
    const int64_t row0 = min((int64_t)qtile * kSQ + wq * kWQ,
                             (p.nq + kQPanel - 1) / kQPanel * kQPanel - kWQ);
    const bool live = (int64_t)qtile * kSQ + wq * kWQ < p.nq;
    const char* qbase = p.Q + row0 / kQPanel * p.q_panel;
    const int qb0 = (int)(row0 % kQPanel) / 16;
    const __amdgpu_buffer_rsrc_t qrs = make_rsrc(reinterpret_cast<const float*>(qbase), p.q_panel);
    const float* qmeta = reinterpret_cast<const float*>(qbase + (int64_t)nk * (kQPanel / 16) * 2 * kFragBytes);
    float qn[QB], iq2[QB];
    int qid[QB];
#pragma unroll
    for (int b = 0; b < QB; ++b) {
        const int q = 16 * (qb0 + b) + col;
        qn[b] = qmeta[q];
        iq2[b] = -2.f * qmeta[kQPanel + q];
        const int64_t row = row0 + 16 * b + col;
        qid[b] = p.qid && row < p.nq ? (int)(p.qid[row] - p.c_base) : -1;
    }

    auto slot_of = [&](auto tag) -> uintx4* {
        constexpr int S = decltype(tag)::value & 3;
        if constexpr (S == 0) return xs0;
        else if constexpr (S == 1) return xs1;
        else if constexpr (S == 2) return xs2;
        else return xs3;
    };
    auto panel_rsrc = [&](int t) {
        return make_rsrc(reinterpret_cast<const float*>(p.C + t * p.c_panel), p.c_panel);
    };
    // stage ks of a centre panel, 16 contiguous kilobytes, straight into LDS
    auto dma = [&](auto tag, __amdgpu_buffer_rsrc_t crs, int ks) {
        uintx4* base = slot_of(tag);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int f = 4 * wave + i;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(crs, (lds_void*)(base + f * 64), 16, lane * 16,
                                                     (ks * 16 + f) * kFragBytes, 0, 0);
        }
    };
    uintx4 bq[2][QB][2];
    auto qload = [&](uintx4 (&b)[QB][2], int ks) {
#pragma unroll
        for (int i = 0; i < QB; ++i)
#pragma unroll
            for (int pl = 0; pl < 2; ++pl)
                b[i][pl] = __builtin_bit_cast(
                    uintx4, __builtin_amdgcn_raw_buffer_load_b128(
                                qrs, lane * 16, (ks * 8 + (qb0 + i) * 2 + pl) * kFragBytes, 0));
    };

    floatx4 sacc[CW][QB];
    floatx4 oacc[LT > 0 ? LT : 1][QB];
#pragma unroll
    for (int c = 0; c < CW; ++c)
#pragma unroll
        for (int b = 0; b < QB; ++b) sacc[c][b] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < LT; ++c)
#pragma unroll
        for (int b = 0; b < QB; ++b) oacc[c][b] = floatx4{0.f, 0.f, 0.f, 0.f};

    [[maybe_unused]] int lolo = 0;                   // low by low products of this panel
    auto step = [&](auto tag, __amdgpu_buffer_rsrc_t crs, int ks) {
        constexpr int S = decltype(tag)::value;
        // the queries' planes change sign here (sign_steps)
        if (ks == p.neg0 || ks == p.neg1) {
#pragma unroll
            for (int c = 0; c < CW; ++c)
#pragma unroll
                for (int i = 0; i < QB; ++i) sacc[c][i] = -sacc[c][i];
        }
        if (ks + 1 < nk) qload(bq[(S & 1) ^ 1], ks + 1);
        if (ks + 3 < nk) dma(std::integral_constant<int, (S + 3) & 3>{}, crs, ks + 3);
        const uintx4* xs = slot_of(tag) + wc * CW * 128;
        const uintx4 (&b)[QB][2] = bq[S & 1];
        uintx4 a[2][2];
        a[0][0] = xs[lane];
        a[0][1] = xs[64 + lane];
#pragma unroll
        for (int c = 0; c < CW; ++c) {
            if (c < CW - 1) {
                a[(c + 1) & 1][0] = xs[(2 * c + 2) * 64 + lane];
                a[(c + 1) & 1][1] = xs[(2 * c + 3) * 64 + lane];
            }
            const uintx4 ah = a[c & 1][0], al = a[c & 1][1];
            if (LL && lolo) {
#pragma unroll
                for (int i = 0; i < QB; ++i) sacc[c][i] = mfma_f16(al, b[i][1], sacc[c][i]);
            }
#pragma unroll
            for (int i = 0; i < QB; ++i) sacc[c][i] = mfma_f16(al, b[i][0], sacc[c][i]);
#pragma unroll
            for (int i = 0; i < QB; ++i) sacc[c][i] = mfma_f16(ah, b[i][1], sacc[c][i]);
#pragma unroll
            for (int i = 0; i < QB; ++i) sacc[c][i] = mfma_f16(ah, b[i][0], sacc[c][i]);
            __builtin_amdgcn_sched_barrier(0);
        }
        // Stage ks + 1 is in LDS for everyone after this barrier without a
        // wait of its own: the products above waited for this step's queries,
        // whose load was issued after dma(ks + 1) (in step ks - 1, which
        // issued dma(ks + 2) after it), and vector-memory operations of a
        // wave complete in order. The scheduling barriers keep the products
        // on this side.
        wg_barrier<-1>();
    };

    auto value = [&](float s, float cn, float ci, int b) {
        // (the scales first: their product overflows only where the distance does)
        return kernel_value<KIND>(fmaf(s, ci * iq2[b], qn[b] + cn), p.scale);
    };

    auto prefetch = [&](int t) {
        const __amdgpu_buffer_rsrc_t crs = panel_rsrc(t);
        dma(std::integral_constant<int, 0>{}, crs, 0);
        if (nk > 1) dma(std::integral_constant<int, 1>{}, crs, 1);
        if (nk > 2) dma(std::integral_constant<int, 2>{}, crs, 2);
        qload(bq[0], 0);
    };
    float4 meta = make_float4(0.f, 0.f, 0.f, 0.f);
    int kp[2] = {-1, -1};
    auto load_meta = [&](int t) {
        if (LL) lolo = __builtin_amdgcn_readfirstlane(p.lolo[t]);
        if (wave == 0)
            meta = *reinterpret_cast<const float4*>(p.C + t * p.c_panel +
                                                    (int64_t)nk * 16 * kFragBytes + lane * 16);
        if (p.kpos) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int64_t c = (int64_t)t * kCPanel + 64 * h + lane;
                kp[h] = c < p.nc ? p.kpos[c] : -1;
            }
        }
    };

    if (t0 < t1) prefetch(t0);
    for (int t = t0; t < t1; ++t) {
        load_meta(t);
        // stages 0..2 are in LDS for everyone; every wave has left the
        // previous tile's epilogue
        wg_barrier<0>();
        if (wave == 0) reinterpret_cast<float4*>(s_meta)[lane] = meta;
        const __amdgpu_buffer_rsrc_t crs = panel_rsrc(t);
        for (int k0 = 0; k0 < nk; k0 += 4) {
            step(std::integral_constant<int, 0>{}, crs, k0);
            if (k0 + 1 < nk) step(std::integral_constant<int, 1>{}, crs, k0 + 1);
            if (k0 + 2 < nk) step(std::integral_constant<int, 2>{}, crs, k0 + 2);
            if (k0 + 3 < nk) step(std::integral_constant<int, 3>{}, crs, k0 + 3);
        }
        if (t + 1 < t1) prefetch(t + 1);
        if (!live) continue;

        // A query's own centre: its distance becomes minus infinity, which
        // the clamp turns into 0 and the kernel value into 1 exactly.
        {
            int rel[QB];
            bool any = false;
#pragma unroll
            for (int b = 0; b < QB; ++b) {
                const int r = qid[b] - t * kCPanel;
                const bool in = qid[b] >= 0 && r >= 0 && r < kCPanel && ((r >> 2) & 3) == g &&
                                (r >> 4) / CW == wc;
                rel[b] = in ? 4 * ((r >> 4) % CW) + (r & 3) : -1;
                any |= in;
            }
            if (__any(any)) {
#pragma unroll
                for (int b = 0; b < QB; ++b)
#pragma unroll
                    for (int c = 0; c < CW; ++c)
#pragma unroll
                        for (int i = 0; i < 4; ++i)
                            if (rel[b] == 4 * c + i) sacc[c][b][i] = __builtin_inff();
            }
        }
        // Subsample centres: their kernel values also go to row kpos of ksb.
        if (p.kpos) {
            const uint64_t f0 = __ballot(kp[0] >= 0), f1 = __ballot(kp[1] >= 0);
            if (f0 | f1) {
#pragma unroll
                for (int c = 0; c < CW; ++c) {
                    const int cc = wc * CW + c;           // block of the panel
                    const unsigned m16 = (unsigned)((cc < 4 ? f0 : f1) >> (16 * (cc & 3))) & 0xffffu;
                    if (!m16) continue;
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        if (!(m16 & (0x1111u << i))) continue;
                        const int at = 16 * cc + 4 * g + i;
                        const int pos = __shfl(cc < 4 ? kp[0] : kp[1], at & 63, 64);
                        const float cn = s_meta[at], ci = s_meta[kCPanel + at];
                        if (pos >= 0) {
                            float* o = p.ksb + pos * p.ldk + row0 + col;
#pragma unroll
                            for (int b = 0; b < QB; ++b) o[16 * b] = value(sacc[c][b][i], cn, ci, b);
                        }
                    }
                }
            }
        }
        [[maybe_unused]] const __amdgpu_buffer_rsrc_t wrs =
            make_rsrc(reinterpret_cast<const float*>(p.W + (int64_t)t * 4 * LT * 3 * kFragBytes),
                      (int64_t)4 * LT * 3 * kFragBytes);
        // (the scheduling barriers keep the compiler from lengthening the
        // weights' lifetimes until they no longer fit the registers)
        [[maybe_unused]] auto load_w = [&](uintx4 (&w)[3], int f) {
#pragma unroll
            for (int pl = 0; pl < 3; ++pl)
                w[pl] = __builtin_bit_cast(uintx4, __builtin_amdgcn_raw_buffer_load_b128(
                                                       wrs, lane * 16, (f * 3 + pl) * kFragBytes, 0));
        };
        [[maybe_unused]] uintx4 wf[2][3];
        const int u0 = wc * (CW / 2);                    // 32-centre groups of this wave
        if constexpr (LT > 0) load_w(wf[0], u0 * LT);
#pragma unroll
        for (int u = 0; u < CW / 2; ++u) {
            uintx4 kf[QB][3];
            const floatx4 cn0 = *reinterpret_cast<const floatx4*>(&s_meta[32 * (u0 + u) + 4 * g]);
            const floatx4 cn1 = *reinterpret_cast<const floatx4*>(&s_meta[32 * (u0 + u) + 16 + 4 * g]);
            const floatx4 ci0 = *reinterpret_cast<const floatx4*>(&s_meta[kCPanel + 32 * (u0 + u) + 4 * g]);
            const floatx4 ci1 = *reinterpret_cast<const floatx4*>(&s_meta[kCPanel + 32 * (u0 + u) + 16 + 4 * g]);
#pragma unroll
            for (int b = 0; b < QB; ++b) {
                float kv[8];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    kv[i] = value(sacc[2 * u][b][i], cn0[i], ci0[i], b);
                    kv[4 + i] = value(sacc[2 * u + 1][b][i], cn1[i], ci1[i], b);
                    if (CW == 2) {                   // see the contraction below
                        kv[i] *= sgn;
                        kv[4 + i] *= sgn;
                    } else if (u & 1) {
                        kv[i] = -kv[i];
                        kv[4 + i] = -kv[4 + i];
                    }
                }
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    unsigned h, m, l;
                    split3(kv[2 * i], kv[2 * i + 1], h, m, l);
                    kf[b][0][i] = h;
                    kf[b][1][i] = m;
                    kf[b][2][i] = l;
                }
                sacc[2 * u][b] = floatx4{0.f, 0.f, 0.f, 0.f};
                sacc[2 * u + 1][b] = floatx4{0.f, 0.f, 0.f, 0.f};
            }
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (LT == 0) {
#pragma unroll
                for (int b = 0; b < QB; ++b) {
                    char* o = p.kplanes + ((row0 / 16 + b) * p.kgroups + 4 * t + u) * 3 * kFragBytes +
                              lane * 16;
#pragma unroll
                    for (int pl = 0; pl < 3; ++pl)
                        *reinterpret_cast<uintx4*>(o + pl * kFragBytes) = kf[b][pl];
                }
            }
#pragma unroll
            for (int j = 0; j < LT; ++j) {
                const int f = u * LT + j;
                if (f + 1 < CW / 2 * LT) load_w(wf[(f + 1) & 1], u0 * LT + f + 1);
                const uintx4 (&w)[3] = wf[f & 1];
                // The products of 32 centres are summed from zero, smallest
                // first, and added to the running sum outside the MFMA, every
                // other time (CW = 2: in every other wave) with both signs
                // turned: an MFMA drops the
                // addends' bits below the accumulator's last places towards
                // minus infinity, which over the thousands of steps of a
                // split shifts every sum the same way (7e-6 of the result at
                // 1.1 million centres in one chain, 1e-6 from zero each time).
                constexpr int wp[6] = {2, 0, 1, 1, 0, 0}, kq[6] = {0, 2, 1, 0, 1, 0};
                floatx4 t[QB];
#pragma unroll
                for (int b = 0; b < QB; ++b) t[b] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int x = 0; x < 6; ++x)
#pragma unroll
                    for (int b = 0; b < QB; ++b) t[b] = mfma_bf16(w[wp[x]], kf[b][kq[x]], t[b]);
#pragma unroll
                for (int b = 0; b < QB; ++b) oacc[j][b] += CW == 2 ? sgn * t[b] : u & 1 ? -t[b] : t[b];
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
    if constexpr (LT > 0 && kCG > 1) {
        // the centre groups' sums, in order, through LDS (the stage slots are
        // free: every wave has passed the last panel's final barrier and no
        // loads into them are in flight)
        floatx4* sum0 = reinterpret_cast<floatx4*>(wq == 0 ? xs0 : xs2);
        floatx4* sum1 = reinterpret_cast<floatx4*>(wq == 0 ? xs1 : xs3);
        static_assert((LT + 1) / 2 * QB * 64 <= kSlotQuads, "half of the sums per slot");
        for (int w = 0; w < kCG; ++w) {
            __syncthreads();
            if (wc == w) {
#pragma unroll
                for (int j = 0; j < LT; ++j)
#pragma unroll
                    for (int b = 0; b < QB; ++b) {
                        floatx4& s = (j & 1 ? sum1 : sum0)[(j / 2 * QB + b) * 64 + lane];
                        if (w > 0) oacc[j][b] = s + oacc[j][b];
                        if (w < kCG - 1) s = oacc[j][b];
                    }
            }
        }
        if (wc != kCG - 1) return;
    }
    if (LT == 0 || !live) return;
    // element i of tile j, block b: label 16 j + 4 g + i, query 16 b + col
    float* o = p.out + ((int64_t)split * p.out_rows + row0) * p.ldw + 4 * g;
#pragma unroll
    for (int b = 0; b < QB; ++b)
#pragma unroll
        for (int j = 0; j < LT; ++j)
            *reinterpret_cast<floatx4*>(o + (int64_t)(16 * b + col) * p.ldw + 16 * j) = oacc[j][b];
}

// ---- contraction of stored kernel values ------------------------------------

// out[q, :] (+)= sum_c K[q, c] W[c, :] over the 32-centre groups of a split,
// from the planes that skmv_kernel<KIND, 0, QB> stored and the planes of W.
// One workgroup = 4 waves owns 128 queries (32 per wave) x 128 labels (8
// tiles). The weights, which the waves share, pass through three LDS slots
// two groups ahead; each wave reads its kernel values from the L2 one group
// ahead. Accumulators for more than 160 labels do not fit beside those of the
// distances, so the kernel values (6 bytes each) make a round trip through
// memory: at 160000 x 2048, 1000 labels, 1601 queries the two launches take
// 2.83 + 2.48 ms, 1.25 PFLOP/s of 16-bit products each, the rate a large
// library product reaches here (one float32 pass: 12.7 ms).
constexpr int kWTiles = 8;                           // label tiles per workgroup
constexpr int kWQ = 128;                             // queries per workgroup
constexpr int kWSlotQuads = kWTiles * 3 * 64;

// wg_barrier for all but the 12 most recent vector-memory operations.
__device__ __forceinline__ void barrier_but_12() {
    asm volatile("s_waitcnt vmcnt(12) lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

__global__ void __launch_bounds__(kSThreads, 2) wmul_kernel(WmulArgs p) {
    __shared__ uintx4 ws0[kWSlotQuads];
    __shared__ uintx4 ws1[kWSlotQuads];
    __shared__ uintx4 ws2[kWSlotQuads];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 15, g = lane >> 4;
    // The label panels of one (query tile, split) share their kernel values,
    // so they run on one XCD (workgroups go to the 8 XCDs round robin).
    const int np = (p.lt + kWTiles - 1) / kWTiles;
    const int tq = (int)((p.nq + kWQ - 1) / kWQ);
    const int item = ((int)blockIdx.x >> 3) / np * 8 + ((int)blockIdx.x & 7);
    const int panel = ((int)blockIdx.x >> 3) % np;
    const int split = item / tq;
    const int qtile = item - split * tq;
    if (split >= p.splits) return;
    const int g0 = (int)min((int64_t)p.groups, split * p.gps);
    const int n = (int)min((int64_t)p.groups, g0 + p.gps) - g0;
    const int nj = min(kWTiles, p.lt - panel * kWTiles);   // label tiles of this panel

    const int64_t row0 = min((int64_t)qtile * kWQ + wave * 32, (p.nq + 31) / 32 * 32 - 32);
    const bool live = (int64_t)qtile * kWQ + wave * 32 < p.nq;
    const char* kbase = p.K + (row0 / 16 * p.kgroups + g0) * 3 * kFragBytes;
    const int64_t kstep = p.kgroups * 3 * kFragBytes;      // next 16 queries
    const char* wbase = p.W + ((int64_t)g0 * p.lt + panel * kWTiles) * 3 * kFragBytes;
    const int64_t wstep = (int64_t)p.lt * 3 * kFragBytes;

    auto slot_of = [&](auto tag) -> uintx4* {
        constexpr int S = decltype(tag)::value % 3;
        if constexpr (S == 0) return ws0;
        else if constexpr (S == 1) return ws1;
        else return ws2;
    };
    auto dma = [&](auto tag, int i) {
        uintx4* base = slot_of(tag);
        const __amdgpu_buffer_rsrc_t wrs =
            make_rsrc(reinterpret_cast<const float*>(wbase + i * wstep), nj * 3 * kFragBytes);
        // (fragments past the panel's last tile read as zero)
#pragma unroll
        for (int f = 0; f < 6; ++f) {
            const int at = 6 * wave + f;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(wrs, (lds_void*)(base + at * 64), 16,
                                                     lane * 16 + at * kFragBytes, 0, 0, 0);
        }
    };
    uintx4 kf[2][2][3];
    auto kload = [&](uintx4 (&k)[2][3], int i) {
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const __amdgpu_buffer_rsrc_t krs = make_rsrc(
                reinterpret_cast<const float*>(kbase + b * kstep + (int64_t)i * 3 * kFragBytes), 3 * kFragBytes);
#pragma unroll
            for (int pl = 0; pl < 3; ++pl)
                k[b][pl] = __builtin_bit_cast(uintx4, __builtin_amdgcn_raw_buffer_load_b128(
                                                          krs, lane * 16, pl * kFragBytes, 0));
        }
    };
    floatx4 oacc[kWTiles][2];
    // element i of tile j, block b: label 16 j + 4 g + i, query 16 b + col
    float* o = p.out + ((int64_t)split * p.out_rows + row0) * p.ldw + panel * kWTiles * 16 + 4 * g;
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int j = 0; j < kWTiles; ++j)
            oacc[j][b] = p.accumulate && j < nj
                             ? *reinterpret_cast<const floatx4*>(o + (int64_t)(16 * b + col) * p.ldw + 16 * j)
                             : floatx4{0.f, 0.f, 0.f, 0.f};

    auto step = [&](auto tag, int i) {
        constexpr int S = decltype(tag)::value;
        if (i + 1 < n) kload(kf[(S + 1) & 1], i + 1);
        if (i + 2 < n) dma(std::integral_constant<int, (S + 2) % 3>{}, i + 2);
        const uintx4* ws = slot_of(tag);
        const uintx4 (&k)[2][3] = kf[S & 1];
        uintx4 w[2][3];
#pragma unroll
        for (int pl = 0; pl < 3; ++pl) w[0][pl] = ws[pl * 64 + lane];
#pragma unroll
        for (int j = 0; j < kWTiles; ++j) {
            if (j >= nj) break;
            if (j + 1 < kWTiles) {
#pragma unroll
                for (int pl = 0; pl < 3; ++pl) w[(j + 1) & 1][pl] = ws[((j + 1) * 3 + pl) * 64 + lane];
            }
            // from zero, smallest first, the sign turned every other group
            // (the stored planes of odd groups are negated): see skmv_kernel
            constexpr int wp[6] = {2, 0, 1, 1, 0, 0}, kq[6] = {0, 2, 1, 0, 1, 0};
            floatx4 t[2] = {floatx4{0.f, 0.f, 0.f, 0.f}, floatx4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
            for (int x = 0; x < 6; ++x)
#pragma unroll
                for (int b = 0; b < 2; ++b) t[b] = mfma_bf16(w[j & 1][wp[x]], k[b][kq[x]], t[b]);
#pragma unroll
            for (int b = 0; b < 2; ++b) oacc[j][b] += S & 1 ? -t[b] : t[b];
        }
        // the next group's weights, fetched a step ago, are in LDS for all
        if (i + 2 < n) barrier_but_12();
        else wg_barrier<0>();
    };
    if (n > 0) {
        dma(std::integral_constant<int, 0>{}, 0);
        if (n > 1) dma(std::integral_constant<int, 1>{}, 1);
        kload(kf[0], 0);
        wg_barrier<0>();
        for (int i = 0; i < n; i += 6) {
            step(std::integral_constant<int, 0>{}, i);
            if (i + 1 < n) step(std::integral_constant<int, 1>{}, i + 1);
            if (i + 2 < n) step(std::integral_constant<int, 2>{}, i + 2);
            if (i + 3 < n) step(std::integral_constant<int, 3>{}, i + 3);
            if (i + 4 < n) step(std::integral_constant<int, 4>{}, i + 4);
            if (i + 5 < n) step(std::integral_constant<int, 5>{}, i + 5);
        }
    }
    if (!live) return;
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int j = 0; j < kWTiles; ++j)
            if (j < nj)
                *reinterpret_cast<floatx4*>(o + (int64_t)(16 * b + col) * p.ldw + 16 * j) = oacc[j][b];
}

typedef void (*SplitFn)(SplitArgs);

template <int KIND, int CW, bool LL>
SplitFn fused_fn(int lt) {
    switch (lt) {
        case 1: return skmv_kernel<KIND, 1, 4, CW, LL>;
        case 2: return skmv_kernel<KIND, 2, 2, CW, LL>;
        case 3: return skmv_kernel<KIND, 3, 2, CW, LL>;
        case 4: return skmv_kernel<KIND, 4, 2, CW, LL>;
        case 5: return skmv_kernel<KIND, 5, 2, CW, LL>;
        case 6: return skmv_kernel<KIND, 6, 2, CW, LL>;
        case 7: return skmv_kernel<KIND, 7, 2, CW, LL>;
        case 8: return skmv_kernel<KIND, 8, 2, CW, LL>;
        case 9: return skmv_kernel<KIND, 9, 2, CW, LL>;
        default: return skmv_kernel<KIND, 10, 2, CW, LL>;
    }
}
template <int KIND, bool LL>
SplitFn kind_fn(int lt, int cw) {
    if (lt == 0) return skmv_kernel<KIND, 0, 4, 8, LL>;
    if (cw == 2) return fused_fn<KIND, 2, LL>(lt);
    if (cw == 4) return fused_fn<KIND, 4, LL>(lt);
    return fused_fn<KIND, 8, LL>(lt);
}
// Kernel for lt label tiles (0: kernel values) and cw blocks per wave.
SplitFn split_fn(int kind, int lt, int cw, bool ll) {
    if (ll) return kind == 0 ? kind_fn<0, true>(lt, cw) : kind_fn<1, true>(lt, cw);
    return kind == 0 ? kind_fn<0, false>(lt, cw) : kind_fn<1, false>(lt, cw);
}

// Queries per workgroup: with one label tile the accumulators leave room for
// four query blocks per wave, else for two.
int split_rows(int64_t lt, int cw) { return (lt <= 1 ? 32 : 16) * cw; }

int split_slots(SplitFn fn) {
    int dev = 0, cus = 256, per = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        cus = 256;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, fn, kSThreads, 0) != hipSuccess || per < 1)
        per = 1;
    return per * cus;
}

}  // namespace

void sign_steps(int64_t nk, int* neg0, int* neg1) {
    *neg0 = *neg1 = -1;
    if (nk < 4) return;
    // the shift grows with the sum: a quarter of the steps, then half with
    // the other sign, then a quarter cancel for a sum growing evenly
    int64_t best = nk * nk;
    for (int64_t a = nk / 4; a <= nk / 4 + 1; ++a)
        for (int64_t b = nk - nk / 4 - 1; b <= nk - nk / 4; ++b) {
            const int64_t off = std::abs(a * a - (b * b - a * a) + (nk * nk - b * b));
            if (a < b && off < best) {
                best = off;
                *neg0 = (int)a;
                *neg1 = (int)b;
            }
        }
}

hipError_t launch_pack_rows(PackArgs a, hipStream_t s) {
    if (a.rows <= 0) return hipSuccess;
    a.nk = feature_steps(a.d);
    a.neg0 = a.neg1 = -1;
    if (a.queries) sign_steps(a.nk, &a.neg0, &a.neg1);
    a.panel = panel_bytes(a.P, a.d);
    const int64_t tiles = round_up(a.rows, a.P) / 16;
    const bool vec = a.d % 4 == 0 && (reinterpret_cast<uintptr_t>(a.X) & 15) == 0;
    // one wave per row where the workgroups alone do not fill the chip (a
    // call of 64 rows of 440 features: 19 us with four waves)
    const dim3 block(tiles < 1024 ? 1024 : 256);
    const dim3 grid(stride_grid(tiles, (int)block.x));
    if (vec) hipLaunchKernelGGL(pack_rows_kernel<true>, grid, block, 0, s, a);
    else hipLaunchKernelGGL(pack_rows_kernel<false>, grid, block, 0, s, a);
    return hipGetLastError();
}

hipError_t launch_pack_weights(const float* W, int64_t rows, int64_t l, int64_t ldw, int64_t lt,
                               void* planes, hipStream_t s) {
    if (rows <= 0) return hipSuccess;
    const int64_t lanes = ceil_div(rows, 32) * lt * 64;
    hipLaunchKernelGGL(pack_weights_kernel, dim3(stride_grid(ceil_div(lanes, 256), 256)), dim3(256), 0,
                       s, W, rows, l, ldw, lt, static_cast<unsigned short*>(planes));
    return hipGetLastError();
}

SplitPlan split_plan(int64_t nq, int64_t nc, int64_t lt, int kind, bool ll, int max_slices) {
    // the fewest centre blocks per wave whose tile still holds all queries
    int cw = 8;
    if (lt > 0)
        while (cw > 2 && split_rows(lt, cw / 2) >= nq) cw /= 2;
    const int64_t slots = split_slots(split_fn(kind, (int)lt, cw, ll));
    const int64_t tq = ceil_div(std::max<int64_t>(nq, 1), split_rows(lt, cw));
    const int64_t nt = ceil_div(std::max<int64_t>(nc, 1), kCPanel);
    SplitPlan best{1, nt, 0.0};
    best.cw = cw;
    double bt = 1e300;
    each_split(nt, max_slices, [&](int64_t P, int64_t per) {
        const double t = (double)ceil_div(tq * P, slots) * ((double)per + 0.5);
        if (t < bt) {
            bt = t;
            best.splits = (int)P;
            best.tps = per;
            best.cost = t;
        }
    });
    return best;
}

SplitPlan wmul_plan(int64_t nq, int64_t groups, int64_t lt, int max_slices) {
    int dev = 0, cus = 256;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        cus = 256;
    const int64_t slots = 2 * (int64_t)cus;          // (launch bounds and LDS)
    const int64_t tiles = ceil_div(std::max<int64_t>(nq, 1), kWQ) * ceil_div(lt, kWTiles);
    const int64_t quads = ceil_div(std::max<int64_t>(groups, 1), 4);
    SplitPlan best{1, 4 * quads, 0.0};
    double bt = 1e300;
    each_split(quads, max_slices, [&](int64_t P, int64_t per) {
        // (partial sums in and out cost about two groups' products)
        const double t = (double)ceil_div(tiles * P, slots) * (4.0 * (double)per + 2.0);
        if (t < bt) {
            bt = t;
            best.splits = (int)P;
            best.tps = 4 * per;
            best.cost = t;
        }
    });
    return best;
}

hipError_t wmul_launch(WmulArgs a, const SplitPlan& p, hipStream_t s) {
    a.splits = p.splits;
    a.gps = p.tps;
    const int64_t items = ceil_div(std::max<int64_t>(a.nq, 1), kWQ) * p.splits;
    hipLaunchKernelGGL(wmul_kernel, dim3((unsigned)(round_up(items, 8) * ceil_div(a.lt, kWTiles))),
                       dim3(kSThreads), 0, s, a);
    return hipGetLastError();
}

hipError_t split_launch(SplitArgs a, const SplitPlan& p, hipStream_t s) {
    a.tps = p.tps;
    sign_steps(a.nk, &a.neg0, &a.neg1);
    const int64_t tq = ceil_div(std::max<int64_t>(a.nq, 1), split_rows(a.lt, p.cw));
    hipLaunchKernelGGL(split_fn(a.kind, a.lt, p.cw, a.lolo != nullptr), dim3((unsigned)(tq * p.splits)),
                       dim3(kSThreads), 0, s, a);
    return hipGetLastError();
}

}  // namespace ep
