// The any-n quantiser: from a weight matrix and per-channel activation statistics to codes,
// per-row lookup tables, group scales and group offsets (any4 paper, section 3.2 "any4
// Algorithm" and appendix, Algorithm 1; scaling equations of section 2.5.1).
//
// Rows are independent, so one block owns one row from start to end and the whole row lives in LDS.
//   1. group-wise scaling: one wavefront per group of 128 weights (two per lane), min / max by
//      wavefront shuffles; alpha, beta are rounded to bf16 first, then w_S = (w - beta) / alpha;
//   2. k-means++ start with the sample weights s = alpha * E|x|: every thread owns a contiguous
//      chunk of the row, chunk masses are scanned across the block, the thread whose chunk holds
//      the drawn point walks it (the uniform draws are an input, one per centre);
//   3. weighted Lloyd iterations in fp64 until a pass changes no code or `iters` centre updates
//      were made, by one of two methods:
//      sorted row (K <= 16384): the scaled row is sorted once (into buckets, whose elements then order themselves; rows
//        that crowd the buckets too much by a bitonic network, 16 elements per thread in registers, LDS between
//        rounds) and running sums of s and s * w_S are kept per 16 sorted elements, a chunk.  A pass is then the work
//        of one wavefront, four lanes per centre: order the centres, find for each neighbouring pair the first sorted
//        position the upper one wins - a search among the chunks' first elements, from where the last pass and the
//        centres' moves let it be expected, that evaluates the very predicate of the E-step (squared fp64 distances,
//        ties to the lower index), then that one chunk - and take every cluster's sums as differences of running sums.
//        The E-step predicate is monotone along the sorted row as long as unequal centres are further apart than the
//        rounding of the distances; a row in which two unequal centres come closer than `centre_gap * max|w_S|`, and
//        one with a NaN or an infinity, is finished by the other method from its starting centres;
//      per weight (larger K, and the rows just named): one pass assigns every weight to its nearest
//        centre and at the same time accumulates, per thread and per centre, sum(s * w_S) and
//        sum(s); the partial sums are combined in a fixed order (lanes, then wavefronts);
//      both are reproducible run to run; they differ from each other (and from a sequential sum)
//      only in the association of the fp64 sums;
//   4. the centres are sorted, the codes renumbered and written with 16-byte stores.
// The sample weights are never stored: s = alpha[group] * act[k] is one fp32 multiply.
#include "any4_device.h"
#include "any4_internal.h"
#include <type_traits>
#include <utility>

#pragma clang fp contract(off)

namespace any4 {

constexpr int QT = 256;                 // threads per block of the per-weight kernel (4 wavefronts; several blocks
                                        // share a compute unit: 512 or 1024 threads measured 1.2 - 2.2x slower)

__device__ __forceinline__ double shfl_xor_f64(double v, int mask) {
    int lo = __double2loint(v), hi = __double2hiint(v);
    lo = __shfl_xor(lo, mask);
    hi = __shfl_xor(hi, mask);
    return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double shfl_up_f64(double v, int delta) {
    int lo = __double2loint(v), hi = __double2hiint(v);
    lo = __shfl_up(lo, delta);
    hi = __shfl_up(hi, delta);
    return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double shfl_f64(double v, int src) {
    int lo = __double2loint(v), hi = __double2hiint(v);
    lo = __shfl(lo, src);
    hi = __shfl(hi, src);
    return __hiloint2double(hi, lo);
}

// f(integral_constant<int, 0>) ... f(integral_constant<int, N - 1>), in order
template <class F, int... I> __device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F> __device__ __forceinline__ void static_for(F&& f) {
    static_for_impl(f, std::make_integer_sequence<int, N>{});
}

// Lane `src` (a constant) of a double, for every lane: two scalar reads, no trip through the LDS pipe.
template <int SRC>
__device__ __forceinline__ double lane_f64(double v) {
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), SRC), __builtin_amdgcn_readlane(__double2loint(v), SRC));
}
// The double `d` lanes down the same row of 16 lanes (0.0 where the row ends): a DPP move per half.
template <int D>
__device__ __forceinline__ double row_shr_f64(double v) {
    return __hiloint2double(__builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x110 + D, 0xF, 0xF, false),
                            __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x110 + D, 0xF, 0xF, false));
}
// The double one lane down (0.0 in lane 0).
__device__ __forceinline__ double wave_shr1_f64(double v) {
    return __hiloint2double(__builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x138, 0xF, 0xF, false),
                            __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x138, 0xF, 0xF, false));
}
// Inclusive sum over the 64 lanes: along the rows of 16 by DPP moves, then the three row totals (scalars)
// onto the rows after them.  A fixed order of additions, like every sum here.
__device__ __forceinline__ double wave_inclusive_sum(double v, int lane) {
    v += row_shr_f64<1>(v);
    v += row_shr_f64<2>(v);
    v += row_shr_f64<4>(v);
    v += row_shr_f64<8>(v);
    const double t0 = lane_f64<15>(v), t1 = lane_f64<31>(v), t2 = lane_f64<47>(v);
    const double o2 = t0 + t1, o3 = o2 + t2;
    const int row = lane >> 4;
    const double off = row == 0 ? 0.0 : row == 1 ? t0 : row == 2 ? o2 : o3;
    return v + off;
}
// min / max over the 64 lanes (the same value in every lane): within rows of 16 by DPP, then four scalars
template <bool MAX>
__device__ __forceinline__ float wave_minmax(float v) {
    auto pick = [](float a, float b) { return MAX ? fmaxf(a, b) : fminf(a, b); };
    auto dpp = [](float x, auto ctrl) {
        return __uint_as_float(__builtin_amdgcn_update_dpp(__float_as_uint(x), __float_as_uint(x), decltype(ctrl)::value, 0xF, 0xF, false));
    };
    v = pick(v, dpp(v, std::integral_constant<int, 0xB1>{}));     // lanes 1 0 3 2 of each four
    v = pick(v, dpp(v, std::integral_constant<int, 0x4E>{}));     // lanes 2 3 0 1
    v = pick(v, dpp(v, std::integral_constant<int, 0x141>{}));    // the half row mirrored
    v = pick(v, dpp(v, std::integral_constant<int, 0x140>{}));    // the row mirrored
    const float a = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(v), 0));
    const float b = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(v), 16));
    const float c = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(v), 32));
    const float d = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(v), 48));
    return pick(pick(a, b), pick(c, d));
}

// ---- 1. group-wise scaling (section 2.5.1): scaled row to ws, group scales to alpha (both LDS)
template <int BITS, int T>
__device__ __forceinline__ void scale_row(const float* __restrict__ wrow, int64_t n, int G, int symmetric,
                                          uint16_t* __restrict__ scale, uint16_t* __restrict__ offset,
                                          float* ws, float* alpha) {
    constexpr int L = 1 << BITS;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const float qrange = symmetric ? (float)((1 << (BITS - 1)) - 1) : (float)(L - 1);
    for (int g = wv; g < G; g += T / kWave) {
        const float2 v = reinterpret_cast<const float2*>(wrow + (int64_t)g * kGroup)[lane];
        const float mn = wave_minmax<false>(fminf(v.x, v.y)), mx = wave_minmax<true>(fmaxf(v.x, v.y));
        const float am = fmaxf(fabsf(mn), fabsf(mx));             // the largest magnitude is at one of the two ends
        const float a32 = symmetric ? am / qrange : (mx - mn) / qrange;
        const float b32 = symmetric ? 0.0f : mn;
        uint32_t ab = f32_to_bf16(a32);
        const uint32_t bb = f32_to_bf16(b32);
        if (bf16_to_f32(ab) == 0.0f) ab = 0x3F80u;                 // constant group: alpha = 1
        const float a = bf16_to_f32(ab), b = bf16_to_f32(bb);
        if (lane == 0) {
            scale[n * G + g] = (uint16_t)ab;
            offset[n * G + g] = (uint16_t)bb;
            alpha[g] = a;
        }
        const float d0 = v.x - b, d1 = v.y - b;
        reinterpret_cast<float2*>(ws + g * kGroup)[lane] = make_float2(d0 / a, d1 / a);
    }
    __syncthreads();
}

template <int BITS, int T>
__device__ __forceinline__ void emit_row_order(const unsigned char* codes, const double* cen, int* misc, int64_t K,
                                               int64_t n, uint8_t* __restrict__ codes_out, uint16_t* __restrict__ lut);

// ---- 3, per weight: Lloyd iterations (E-step: nearest centre; M-step: Eq. (B), weighted mean) over ws in row
// order, then 4: sorted centres, renumbered codes, stores.  cen holds the starting centres.
template <int BITS, int T>
__device__ __forceinline__ void lloyd_per_weight(const float* ws, unsigned char* codes, const float* alpha, double* red,
                                                 double* cen, int* misc, const float* __restrict__ act, int64_t K,
                                                 int iters, int64_t n, uint8_t* __restrict__ codes_out,
                                                 uint16_t* __restrict__ lut, int32_t* __restrict__ msteps) {
    constexpr int L = 1 << BITS;
    constexpr int W = T / kWave;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    auto sample_weight = [&](int j) -> float { return alpha[j >> 7] * (act ? act[j] : 1.0f); };
    for (int j = tid; j < K; j += T) codes[j] = 0xFF;
    int done = 0;
    for (;;) {
        double c[L];
#pragma unroll
        for (int p = 0; p < L; ++p) c[p] = cen[p];
        double num[L], den[L];
#pragma unroll
        for (int p = 0; p < L; ++p) { num[p] = 0.0; den[p] = 0.0; }
        int changed = 0;
#pragma unroll 2                                               // two independent chains of compare / select: 5 % faster
        for (int j = tid; j < K; j += T) {
            const double x = (double)ws[j];
            int best = 0;
            double bd = (x - c[0]) * (x - c[0]);
#pragma unroll
            for (int p = 1; p < L; ++p) {
                const double d = x - c[p];
                const double dd = d * d;
                if (dd < bd) { bd = dd; best = p; }
            }
            changed |= (codes[j] != (unsigned char)best);
            codes[j] = (unsigned char)best;
            const double s = (double)sample_weight(j);
            const double sx = s * x;
            // num[best] += sx, den[best] += s with the accumulators in registers: one fused multiply-add
            // per accumulator with a factor of exactly 1 or 0 (fma(v, 1, a) = a + v rounded once;
            // fma(v, 0, a) = a), cheaper than selecting v or 0 and adding
#pragma unroll
            for (int p = 0; p < L; ++p) {
                const double one = __hiloint2double(best == p ? 0x3FF00000 : 0, 0);
                num[p] = __builtin_fma(sx, one, num[p]);
                den[p] = __builtin_fma(s, one, den[p]);
            }
        }
        changed = __syncthreads_or(changed);
        if ((done > 0 && !changed) || done >= iters) break;
        // combine the partial sums: butterfly over the lanes, then the wavefronts in order
#pragma unroll
        for (int p = 0; p < L; ++p) {
#pragma unroll
            for (int m = 1; m < 64; m <<= 1) {
                num[p] += shfl_xor_f64(num[p], m);
                den[p] += shfl_xor_f64(den[p], m);
            }
        }
        if (lane == 0) {
#pragma unroll
            for (int p = 0; p < L; ++p) { red[(wv * 2 + 0) * L + p] = num[p]; red[(wv * 2 + 1) * L + p] = den[p]; }
        }
        __syncthreads();
        if (tid < L) {
            double a = 0.0, b = 0.0;
            for (int i = 0; i < W; ++i) { a += red[(i * 2 + 0) * L + tid]; b += red[(i * 2 + 1) * L + tid]; }
            if (b > 0.0) cen[tid] = a / b;
        }
        ++done;
        __syncthreads();
    }
    if (msteps && tid == 0) msteps[n] = done;
    emit_row_order<BITS, T>(codes, cen, misc, K, n, codes_out, lut);
}

// The same iterations for the rarely taken hand-over inside the sorted-row kernel, which has 128 registers per lane: the
// E-step and the M-step are separate passes, so that the centres and the accumulators are never in registers together.
// Every accumulator still adds its weights in the same order, so the sums are the same bit for bit.  A short row has one or
// two wavefronts, and a chip with few rows nothing else to do meanwhile: what counts is latency, so the E-step carries
// four weights at a time and the M-step loads two before it adds them, once for all centres.  All rows handed over, any4,
// against one weight at a time and four centres per sweep: 512 x 1024 568 -> 281 us (in blocks of four wavefronts, as
// for longer rows, 372 with the slower loops), 512 x 2048 678 -> 378, 6144 x 4096 5250 -> 3670, 256 x 14336 967 -> 738.
template <int BITS, int T>
__device__ __forceinline__ void lloyd_per_weight_lean(const float* ws, unsigned char* codes, const float* alpha, double* red,
                                                   double* cen, int* misc, const float* __restrict__ act, int K,
                                                   int iters, int64_t n, uint8_t* __restrict__ codes_out,
                                                   uint16_t* __restrict__ lut, int32_t* __restrict__ msteps) {
    constexpr int L = 1 << BITS;
    constexpr int W = T / kWave;
    constexpr int E = 4, M = 2;
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    for (int j = tid; j < K; j += T) codes[j] = 0xFF;
    __syncthreads();
    int done = 0;
    for (;;) {
        int changed = 0;
        if (tid == 0) misc[40] = 0;                                // "some code changed in this pass"
        __syncthreads();
        {
            double c[L];
#pragma unroll
            for (int p = 0; p < L; ++p) c[p] = cen[p];
#pragma unroll 1
            for (int j = tid; j < K; j += E * T) {
                double x[E], bd[E];
                int best[E], was[E];
#pragma unroll
                for (int k = 0; k < E; ++k) {
                    const int jk = min(j + k * T, K - 1);          // (past the row: nothing is stored)
                    x[k] = (double)ws[jk];
                    was[k] = codes[jk];
                    bd[k] = (x[k] - c[0]) * (x[k] - c[0]);
                    best[k] = 0;
                }
#pragma unroll
                for (int p = 1; p < L; ++p) {
#pragma unroll
                    for (int k = 0; k < E; ++k) {
                        const double d = x[k] - c[p];
                        const double dd = d * d;
                        if (dd < bd[k]) { bd[k] = dd; best[k] = p; }
                    }
                }
#pragma unroll
                for (int k = 0; k < E; ++k) {
                    if (j + k * T < K) {
                        changed |= was[k] != best[k];
                        codes[j + k * T] = (unsigned char)best[k];
                    }
                }
            }
        }
        if (changed) misc[40] = 1;
        __syncthreads();
        changed = misc[40];
        if ((done > 0 && !changed) || done >= iters) break;
        {
            double num[L], den[L];
#pragma unroll
            for (int p = 0; p < L; ++p) { num[p] = 0.0; den[p] = 0.0; }
#pragma unroll 1
            for (int j = tid; j < K; j += M * T) {
                float x[M], s[M];
                int best[M];
#pragma unroll
                for (int k = 0; k < M; ++k) {
                    const int jk = j + k * T;
                    const bool in = jk < K;                        // (past the row: adds 0 * 0)
                    x[k] = in ? ws[jk] : 0.0f;
                    s[k] = in ? alpha[jk >> 7] * (act ? act[jk] : 1.0f) : 0.0f;
                    best[k] = in ? (int)codes[jk] : 0;
                }
#pragma unroll
                for (int k = 0; k < M; ++k) {
                    const double sd = (double)s[k], sx = sd * (double)x[k];
#pragma unroll
                    for (int p = 0; p < L; ++p) {
                        const double one = __hiloint2double(best[k] == p ? 0x3FF00000 : 0, 0);
                        num[p] = __builtin_fma(sx, one, num[p]);
                        den[p] = __builtin_fma(sd, one, den[p]);
                    }
                }
            }
#pragma unroll
            for (int p = 0; p < L; ++p) {
#pragma unroll
                for (int m = 1; m < 64; m <<= 1) {
                    num[p] += shfl_xor_f64(num[p], m);
                    den[p] += shfl_xor_f64(den[p], m);
                }
                if (lane == 0) { red[(wv * 2 + 0) * L + p] = num[p]; red[(wv * 2 + 1) * L + p] = den[p]; }
            }
        }
        __syncthreads();
        if (tid < L) {
            double a = 0.0, b = 0.0;
#pragma unroll 1
            for (int i = 0; i < W; ++i) { a += red[(i * 2 + 0) * L + tid]; b += red[(i * 2 + 1) * L + tid]; }
            if (b > 0.0) cen[tid] = a / b;
        }
        ++done;
        __syncthreads();
    }
    if (msteps && tid == 0) msteps[n] = done;
    emit_row_order<BITS, T>(codes, cen, misc, K, n, codes_out, lut);
}

// ---- 4, per weight: sort the centres (stable), renumber the codes (LDS, row order), store
template <int BITS, int T>
__device__ __forceinline__ void emit_row_order(const unsigned char* codes, const double* cen, int* misc, int64_t K,
                                               int64_t n, uint8_t* __restrict__ codes_out, uint16_t* __restrict__ lut) {
    constexpr int L = 1 << BITS;
    const int tid = threadIdx.x;
    __syncthreads();
    if (tid == 0) {
        int* order = misc + 1 + L;
        for (int p = 0; p < L; ++p) order[p] = p;
        for (int i = 1; i < L; ++i) {
            const int o = order[i];
            int p = i;
            while (p > 0 && cen[order[p - 1]] > cen[o]) { order[p] = order[p - 1]; --p; }
            order[p] = o;
        }
        for (int r = 0; r < L; ++r) {
            misc[1 + order[r]] = r;
            lut[n * L + r] = (uint16_t)f32_to_bf16((float)cen[order[r]]);
        }
    }
    __syncthreads();
    unsigned long long rank = 0;                                  // rank of centre p in nibble p
    for (int p = 0; p < L; ++p) rank |= (unsigned long long)misc[1 + p] << (4 * p);
    uint8_t* crow = codes_out + n * K;
    for (int j = tid * 16; j < K; j += T * 16) {
        uint4 v = *reinterpret_cast<const uint4*>(codes + j);
        uint32_t in[4] = {v.x, v.y, v.z, v.w}, out[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            uint32_t o = 0;
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                const uint32_t code = (in[i] >> (8 * b)) & 0xFFu;
                o |= (uint32_t)((rank >> (4 * code)) & 0xFull) << (8 * b);
            }
            out[i] = o;
        }
        *reinterpret_cast<uint4*>(crow + j) = make_uint4(out[0], out[1], out[2], out[3]);
    }
}

// =====================================================================================================
// The per-weight kernel (any K up to the LDS limit).
// LDS of one block: ws [K] f32 | codes [K] u8 | alpha [K/128] f32 (padded to 16 B) | scan [W] f64 |
// red [W][2][L] f64 | cen [L] f64 | misc [64] i32
constexpr size_t quantize_small_offset(int64_t K) {
    return ((size_t)K * 5 + (size_t)(K / kGroup) * 4 + 15) & ~(size_t)15;
}
constexpr size_t quantize_lds_bytes(int64_t K, int bits) {
    return quantize_small_offset(K) + (size_t)(QT / kWave) * 8 + (size_t)(QT / kWave) * 2 * (1 << bits) * 8 +
           (size_t)(1 << bits) * 8 + 64 * 4;
}

template <int BITS>
__global__ __launch_bounds__(QT) void quantize_kernel(
    const float* __restrict__ w, const float* __restrict__ act, const float* __restrict__ u,
    int64_t K, int symmetric, int iters, uint8_t* __restrict__ codes_out, uint16_t* __restrict__ lut,
    uint16_t* __restrict__ scale, uint16_t* __restrict__ offset, int32_t* __restrict__ msteps) {
    constexpr int L = 1 << BITS;
    constexpr int QW = QT / kWave;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int G = (int)(K / kGroup);
    float* ws = reinterpret_cast<float*>(smem);
    unsigned char* codes = smem + (size_t)K * 4;
    float* alpha = reinterpret_cast<float*>(smem + (size_t)K * 5);
    double* scan = reinterpret_cast<double*>(smem + quantize_small_offset(K));     // [QW]
    double* red = scan + QW;                     // [QW][2][L]
    double* cen = red + QW * 2 * L;              // [L]
    int* misc = reinterpret_cast<int*>(cen + L); // [0] selected index, [1 .. L] rank of a centre, [1 + L .. 2L] sort order

    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int64_t n = blockIdx.x;
    scale_row<BITS, QT>(w + n * K, n, G, symmetric, scale, offset, ws, alpha);

    auto sample_weight = [&](int j) -> float { return alpha[j >> 7] * (act ? act[j] : 1.0f); };

    // ---- 2. k-means++ with sample weights; thread t owns the chunk [t * C, (t + 1) * C)
    const int C = (int)((K + QT - 1) / QT);
    const int j0 = min(tid * C, (int)K), j1 = min(j0 + C, (int)K);
    for (int q = 0; q < L; ++q) {
        // mass of a sample: s for the first centre, s * (squared distance to the nearest chosen centre) after
        auto mass = [&](int j) -> double {
            const double s = (double)sample_weight(j);
            if (q == 0) return s;
            const double x = (double)ws[j];
            double best = (x - cen[0]) * (x - cen[0]);
            for (int p = 1; p < q; ++p) {
                const double d = x - cen[p];
                const double dd = d * d;
                if (dd < best) best = dd;
            }
            return s * best;
        };
        double part = 0.0;
        for (int j = j0; j < j1; ++j) part += mass(j);
        // inclusive scan of the chunk masses over the block: lanes, then wavefronts
        double inc = part;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const double o = shfl_up_f64(inc, d);
            if (lane >= d) inc += o;
        }
        if (lane == 63) scan[wv] = inc;
        __syncthreads();
        double base = 0.0;
        for (int i = 0; i < wv; ++i) base += scan[i];
        double total = 0.0;
        for (int i = 0; i < QW; ++i) total += scan[i];
        inc += base;
        // running mass at the end of the previous chunk: the neighbour's own value, so that the
        // chunks' intervals [before, inc) tile [0, total) without gaps
        double before = shfl_up_f64(inc, 1);
        if (lane == 0) before = base;
        if (tid == 0) misc[0] = 0x7FFFFFFF;
        __syncthreads();
        if (total > 0.0) {
            const double t = (double)u[n * L + q] * total;
            // the first chunk whose running mass exceeds t holds the drawn sample
            if (before <= t && inc > t && j0 < j1) {
                double run = before;
                int pick = -1, lastpos = j0;
                for (int j = j0; j < j1; ++j) {
                    const double m = mass(j);
                    run += m;
                    if (m > 0.0) lastpos = j;
                    if (run > t) { pick = j; break; }
                }
                atomicMin(&misc[0], pick >= 0 ? pick : lastpos);
            }
        } else if (tid == 0) {
            int64_t j = (int64_t)((double)u[n * L + q] * (double)K);
            misc[0] = (int)min(j, K - 1);
        }
        __syncthreads();
        int sel = misc[0];
        if (sel >= K) sel = (int)K - 1;       // not reachable with finite, non-negative masses
        if (tid == 0) cen[q] = (double)ws[sel];
        __syncthreads();
    }

    lloyd_per_weight<BITS, QT>(ws, codes, alpha, red, cen, misc, act, K, iters, n, codes_out, lut, msteps);
}

// =====================================================================================================
// The sorted-row kernel.  T threads sort KP = 16 T elements (K <= KP; the tail is padding that sorts last).
//
// LDS of one block (PADW = KP + KP / 16 elements: one spare element after every 16 keeps all three access
// patterns of the sort - 16 neighbours per thread, strides of 16, strides of 256 - off each other's banks):
//   kv [PADW] u32 x 2   the row's scaled weights (fp32, row order, in the first 4 K bytes) until the sort; then
//                       the elements (order-preserving integer image of w_S, sample weight s as fp32 bits),
//                       ascending in w_S.  (The per-weight method keeps its codes behind the scaled weights.)
//   alpha [KP/128] f32 | pre_s, pre_sx [T + 1] f64 (running sums before every 16th sorted element; the total)
//   scan [2 W] f64 | cen [L] f64 | cen0 [L] f64 | misc [44] i32
//   (the per-weight method's partial sums red [W][2][L] f64 lie over pre_s: 2 W L <= 2 (T + 1); the smallest key of the cluster
//   of rank i, fin [L] u32, over cen, which the sorted row's passes read only once)
// A compute unit holds 16 wavefronts of this kernel by their registers, and as many by its LDS: 16 blocks of one wavefront
// have 10240 bytes each (with 10368, and fewer blocks, 11525 x 1024 any4 took 256 us; 243).
constexpr int kSortedMaxK = 16384;
constexpr size_t sorted_padw(int T) { return (size_t)T * 17; }
constexpr size_t sorted_lds_bytes(int T, int bits) {
    const size_t W = (size_t)T / kWave, L = (size_t)1 << bits;
    return sorted_padw(T) * 8 + ((size_t)T / 8) * 4 + 2 * ((size_t)T + 1) * 8 + 2 * W * 8 + 2 * L * 8 + 44 * 4;
}
constexpr bool sorted_blocks_fit(int T) { return sorted_lds_bytes(T, 4) <= (size_t)160 * 1024 * T / (16 * kWave); }
static_assert(sorted_blocks_fit(64) && sorted_blocks_fit(128) && sorted_blocks_fit(256) && sorted_blocks_fit(512) && sorted_blocks_fit(1024));

__device__ __forceinline__ int pad16(int p) { return p + (p >> 4); }
// fp32 -> u32 whose unsigned order is the order of the numbers (finite inputs), and back
__device__ __forceinline__ uint32_t f32_key(float f) {
    const uint32_t b = __float_as_uint(f);
    return b ^ ((b >> 31) ? 0xFFFFFFFFu : 0x80000000u);
}
__device__ __forceinline__ float key_f32(uint32_t k) {
    return __uint_as_float(k ^ ((k >> 31) ? 0x80000000u : 0xFFFFFFFFu));
}
constexpr uint32_t kPadKey = 0xFFFFFFFFu;         // sorts after every number; its sample weight is 0

// Compare-exchange of two elements (key, sample weight): the smaller key goes to the first.
// (The empty asm statement keeps the two sample weights plain values: left alone, the compiler turns
// "one or the other element of the array" into an element picked by a computed index, which costs a
// chain of 16 selects per compare-exchange.)
__device__ __forceinline__ void compare_exchange(uint32_t& k1, uint32_t& s1, uint32_t& k2, uint32_t& s2) {
    uint32_t a = s1, b = s2;
    asm("" : "+v"(a), "+v"(b));
    const bool sw = k1 > k2;
    const uint32_t ka = min(k1, k2), kb = max(k1, k2);
    s1 = sw ? b : a;
    s2 = sw ? a : b;
    k1 = ka;
    k2 = kb;
}

// The first four merge sizes (2 .. 16) of the bitonic network stay inside the 16 neighbouring elements
// of a thread: one trip through LDS.  Up to size 8 the direction of a pair is a bit of its place among
// the 16 (known when compiling: descending = the roles swapped); for size 16 it is the thread's parity.
template <int T>
__device__ __forceinline__ void sort_first16(uint2* kv) {
    int base = threadIdx.x * 17;
    asm volatile("" : "+v"(base));
    uint32_t kk[16], ss[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const uint2 v = kv[base + r];
        kk[r] = v.x;
        ss[r] = v.y;
    }
#pragma unroll
    for (int m = 1; m <= 4; ++m) {
        const uint32_t flip = m == 4 ? (uint32_t)(-(int)(threadIdx.x & 1)) : 0u;
        if (m == 4) {
#pragma unroll
            for (int r = 0; r < 16; ++r) kk[r] ^= flip;
        }
#pragma unroll
        for (int b = m - 1; b >= 0; --b) {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                if ((r & (1 << b)) != 0) continue;
                const int r2 = r | (1 << b);
                if (m < 4 && ((r >> m) & 1)) compare_exchange(kk[r2], ss[r2], kk[r], ss[r]);
                else compare_exchange(kk[r], ss[r], kk[r2], ss[r2]);
            }
        }
        if (m == 4) {
#pragma unroll
            for (int r = 0; r < 16; ++r) kk[r] ^= flip;
        }
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) kv[base + r] = make_uint2(kk[r], ss[r]);
    __syncthreads();
}

// One round of the bitonic network on the 16 elements a thread holds: the elements differ in bits
// WB .. WB + NB - 1 of their position (16 / 2^NB independent groups per thread); the round runs the
// compare-exchange stages of merge size 2^m (m > top) for the strides 2^top .. 2^WB.  Pairs that sort
// descending (bit m of the position set) have their keys complemented on the way in and out, so that every
// compare-exchange is the same ascending one.  With the spare element after every 16, the 2^NB elements
// of a group lie a fixed distance apart.
template <int T, int WB, int NB>
__device__ __forceinline__ void sort_round(uint2* kv, int m, int top) {
    constexpr int E = 1 << NB, GROUPS = 16 / E;
    constexpr int STRIDE = WB >= 4 ? (1 << WB) + (1 << (WB >= 4 ? WB - 4 : 0)) : 1;
    // (the empty asm statement ties the addresses to this call: computed once for all calls, outside the
    // loop over the merge sizes, they would hold registers through the whole sort)
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    const bool inside = m < WB + NB;                   // the direction bit is one of the bits the 2^NB elements differ in
    uint32_t kk[16], ss[16], flip[16];
    int base[GROUPS];
#pragma unroll
    for (int g = 0; g < GROUPS; ++g) {
        const int low = g * T + tid;
        const int pos0 = ((low >> WB) << (WB + NB)) | (low & ((1 << WB) - 1));
        base[g] = pos0 + (pos0 >> 4);
        const uint32_t gflip = inside ? 0u : (uint32_t)(-(int)(((uint32_t)low >> (m - NB)) & 1u));
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int r = g * E + e;
            const uint32_t eflip = inside ? (uint32_t)(-(int)(((uint32_t)e >> (m - WB)) & 1u)) : 0u;   // the same in all lanes
            flip[r] = gflip | eflip;
            const uint2 v = kv[base[g] + e * STRIDE];
            kk[r] = v.x ^ flip[r];
            ss[r] = v.y;
        }
    }
#pragma unroll
    for (int b = NB - 1; b >= 0; --b) {
        if (WB + b > top) continue;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            if ((r & (1 << b)) != 0) continue;
            const int r2 = r | (1 << b);
            compare_exchange(kk[r], ss[r], kk[r2], ss[r2]);
        }
    }
#pragma unroll
    for (int g = 0; g < GROUPS; ++g)
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int r = g * E + e;
            kv[base[g] + e * STRIDE] = make_uint2(kk[r] ^ flip[r], ss[r]);
        }
    __syncthreads();
}

// Inclusive sum of a u32 over the 64 lanes, min / max of a u32 over the 64 lanes (in every lane).
__device__ __forceinline__ uint32_t wave_inclusive_sum_u32(uint32_t v, int lane) {
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x111, 0xF, 0xF, false);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x112, 0xF, 0xF, false);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x114, 0xF, 0xF, false);
    v += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x118, 0xF, 0xF, false);
    const uint32_t t0 = __builtin_amdgcn_readlane(v, 15), t1 = __builtin_amdgcn_readlane(v, 31), t2 = __builtin_amdgcn_readlane(v, 47);
    const int row = lane >> 4;
    return v + (row == 0 ? 0u : row == 1 ? t0 : row == 2 ? t0 + t1 : t0 + t1 + t2);
}
template <bool MAX>
__device__ __forceinline__ uint32_t wave_minmax_u32(uint32_t v) {
    auto pick = [](uint32_t a, uint32_t b) { return MAX ? max(a, b) : min(a, b); };
    auto dpp = [](uint32_t x, auto ctrl) { return (uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)x, decltype(ctrl)::value, 0xF, 0xF, false); };
    v = pick(v, dpp(v, std::integral_constant<int, 0xB1>{}));
    v = pick(v, dpp(v, std::integral_constant<int, 0x4E>{}));
    v = pick(v, dpp(v, std::integral_constant<int, 0x141>{}));
    v = pick(v, dpp(v, std::integral_constant<int, 0x140>{}));
    const uint32_t a = __builtin_amdgcn_readlane(v, 0), b = __builtin_amdgcn_readlane(v, 16);
    const uint32_t c = __builtin_amdgcn_readlane(v, 32), d = __builtin_amdgcn_readlane(v, 48);
    return pick(pick(a, b), pick(c, d));
}

// `n`, and one more if element `o` comes before `me` in the order (key, sample weight, place in the bucket), where its place
// less PLACE is `d` below that of `me`: one borrow carried through the three words, four instructions at full rate (a
// comparison of 64-bit integers is not one).
template <int PLACE>
__device__ __forceinline__ uint32_t count_below(uint32_t n, uint2 o, uint2 me, int d) {
    uint32_t t;
    asm("v_cmp_lt_i32_e32 vcc, %6, %7\n\t"
        "v_subb_co_u32_e32 %1, vcc, %2, %3, vcc\n\t"
        "v_subb_co_u32_e32 %1, vcc, %4, %5, vcc\n\t"
        "v_addc_co_u32_e32 %0, vcc, 0, %0, vcc"
        : "+v"(n), "=&v"(t) : "v"(o.y), "v"(me.y), "v"(o.x), "v"(me.x), "n"(PLACE), "v"(d) : "vcc");
    return n;
}

// Sort by distribution: 32 T buckets of equal width between the row's smallest and largest scaled weight, filled by a
// counting sort (two 16-bit counters to a word of LDS); then every element counts the smaller ones of its bucket.
// Group scaling spreads a row over a fixed range, so most buckets hold about one element, and the sort is ~1.5 k
// instructions per thread where the bitonic network of 16 T elements takes ~8 k (K <= 4096) to ~11 k.  The order among
// the elements of a bucket is (key, sample weight): the sorted row does not depend on the order in which the counters
// were bumped.  Bound: LDS latency and vector issue.  Against the network, fp32 weights: 6144 x 4096 any4 836 -> 698 us for
// the whole kernel, of which the sort was 78 then; 4096 x 14336 2704 -> 2070 us, the sort 275 of it.
// Equal weights crowd a bucket.  Weights that are bf16 numbers do so by nature: the offset is a group's smallest weight
// itself, which scales to exactly 0, once a group at least (112 - 130 in a row of 14336), and pruned weights are equal
// within a group.  The elements of a bucket of more than kBucketOwn go on a list and are ranked from there by four lanes
// each: left with their owners, a few of them in a wavefront make all its lanes go round the bucket.  The list is as
// large as the LDS that is free here, 4 T elements; a row with more takes it in several rounds.  bf16 weights, the network
// (what they had when a bucket of more than 32 sent a row there) against the list: 4096 x 14336 2055 -> 1461 us (fp32 1386),
// 4096 x 8192 904 -> 654, 6144 x 4096 591 -> 502; half of 4096 x 14336 pruned 2159 -> 1920.
// False, and nothing sorted, where the buckets would not do: all weights equal, a weight that is not finite, a bucket of
// more than kBucketMost (what a slot has bits for), or a list that costs more than the network.  Its cost is counted in
// looks, the squares of the sizes of its buckets.  The network wins from 46 looks per weight of the row on where equal
// weights are neighbours, whose threads look at the same elements, and from 25 on where they lie scattered over the row
// (4096 x 14336; at K = 1024 .. 4096 from 35 - 44 and from 20 - 25).  Equal scaled weights are mostly of one group, and half of
// the weights pruned make 32 - 44, so kBucketLooks is at the former; a row of 352 scattered values, 40 weights each, 39
// looks per weight, pays for it (2286 us against 1775).  Sizes from 8 to 24 as kBucketOwn time alike.
// `key`, `sv`: the 16 elements of a thread that has any (`mine`); scratch: `scan` 4 W words, `list` 4 T words, `flag` one and
// `count` two.  LDS of kv is free on entry once every thread has arrived.
constexpr uint32_t kBucketOwn = 16;
constexpr uint32_t kBucketMost = 512;
constexpr uint32_t kBucketLooks = 44;             // per weight of the row
template <int T>
__device__ __forceinline__ bool sort_by_buckets(uint2* kv, uint32_t* scan, uint32_t* list, int* flag, int* count,
                                                const uint32_t (&key)[16], const float (&sv)[16], bool mine, int K) {
    constexpr int W = T / kWave;
    constexpr int NB = 32 * T, LIST = 4 * T;
    static_assert(16 * T <= 1 << 14 && kBucketMost <= 512, "an element's slot: 14 bits of position, 9 of its bucket's size, 9 of its place");
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));
    uint32_t lo = 0xFFFFFFFFu, hi = 0u;
#pragma unroll
    for (int e = 0; e < 16; ++e) { lo = min(lo, key[e]); hi = max(hi, key[e]); }
    lo = mine ? lo : 0xFFFFFFFFu;
    hi = mine ? hi : 0u;
    lo = wave_minmax_u32<false>(lo);
    hi = wave_minmax_u32<true>(hi);
    if (lane == 0) { scan[2 * wv] = lo; scan[2 * wv + 1] = hi; }
    if (tid == 0) { *flag = 0; count[0] = count[1] = 0; }
    __syncthreads();                                               // every thread is done with what lay in kv
    uint32_t* const hist = reinterpret_cast<uint32_t*>(kv);        // [NB / 2] words, and one counter more
#pragma unroll 1
    for (int i = 0; i < W; ++i) { lo = min(lo, scan[2 * i]); hi = max(hi, scan[2 * i + 1]); }
    const float mn = key_f32(lo), range = key_f32(hi) - mn;
    // (not finite: a NaN or an infinity among the weights, or a range beyond fp32)
    if (!(range > 0.0f && range < __uint_as_float(0x7F800000u)) || !(fabsf(mn) < __uint_as_float(0x7F800000u))) return false;   // the same in every thread
    const float inv = (float)NB / range;
    if (!(inv < __uint_as_float(0x7F800000u))) return false;
#pragma unroll
    for (int i = 0; i < 4; ++i) reinterpret_cast<uint4*>(hist)[i * T + tid] = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
    // bucket (monotone in the weight: one subtraction, one product, both rounded monotonically) and place in it
    uint32_t slot[16] = {}, rmax = 0;
    if (mine) {
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const uint32_t b = (uint32_t)__builtin_amdgcn_fmed3f((key_f32(key[e]) - mn) * inv, 0.0f, (float)(NB - 1));
            const uint32_t old = atomicAdd(&hist[b >> 1], (b & 1) ? 0x10000u : 1u);
            const uint32_t r = (b & 1) ? old >> 16 : old & 0xFFFFu;
            rmax = max(rmax, r);
            slot[e] = b | (r << 16);
        }
        if (rmax >= kBucketMost) *flag = 1;
    }
    if (__ballot(rmax >= kBucketOwn) != 0ull) {
        // squares of the sizes of the buckets with more than kBucketOwn elements, by the places in them
        uint32_t looks = 0;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const uint32_t r = slot[e] >> 16;
            looks += r > kBucketOwn ? 2 * r + 1 : r == kBucketOwn ? (r + 1) * (r + 1) : 0u;
        }
        looks = wave_inclusive_sum_u32(looks, lane);
        if (lane == 63) atomicAdd(count + 1, (int)looks);
    }
    __syncthreads();
    if (*flag != 0 || (uint32_t)count[1] > kBucketLooks * (uint32_t)K) return false;
    // counters -> first position of every bucket; a thread has 32 neighbouring ones
    {
        uint32_t c[16], sum = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint4 v = reinterpret_cast<const uint4*>(hist)[tid * 4 + i];
            c[4 * i] = v.x; c[4 * i + 1] = v.y; c[4 * i + 2] = v.z; c[4 * i + 3] = v.w;
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) sum += (c[i] & 0xFFFFu) + (c[i] >> 16);
        uint32_t run = wave_inclusive_sum_u32(sum, lane);
        if (lane == 63) scan[2 * W + wv] = run;
        run -= sum;
        __syncthreads();
#pragma unroll 1
        for (int i = 0; i < wv; ++i) run += scan[2 * W + i];
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const uint32_t second = run + (c[i] & 0xFFFFu), next = second + (c[i] >> 16);
            c[i] = run | (second << 16);
            run = next;
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
            reinterpret_cast<uint4*>(hist)[tid * 4 + i] = make_uint4(c[4 * i], c[4 * i + 1], c[4 * i + 2], c[4 * i + 3]);
        if (tid == T - 1) hist[NB / 2] = run;                      // = K
    }
    __syncthreads();
    // first position, size less one of the element's bucket, and its place in it
    const uint16_t* const first = reinterpret_cast<const uint16_t*>(hist);
    uint32_t most = 0;
    if (mine) {
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const uint32_t b = slot[e] & 0xFFFFu, r = slot[e] >> 16;
            const uint32_t f = first[b], size = first[b + 1] - f;
            slot[e] = f | ((size - 1) << 14) | (r << 23);
            most = max(most, size);
        }
    }
    __syncthreads();
    // into the buckets (no spare elements yet), and what sorts last behind the row: a look beyond a bucket's end
    // finds larger keys only
    auto position = [](uint32_t s) { return s & 0x3FFFu; };
    auto bucket_size = [](uint32_t s) { return ((s >> 14) & 0x1FFu) + 1; };
    auto place = [](uint32_t s) { return s >> 23; };
    if (mine) {
#pragma unroll
        for (int e = 0; e < 16; ++e) kv[position(slot[e]) + place(slot[e])] = make_uint2(key[e], __float_as_uint(sv[e]));
    }
    if (tid < 16) kv[K + tid] = make_uint2(kPadKey, 0u);
    most = wave_minmax_u32<true>(most);
    uint32_t waiting = 0, listed = 0;                              // bit e: element e is to go on the list; is or was on it
    auto put = [&]() {
        const uint32_t n = (uint32_t)__popc(waiting), to = wave_inclusive_sum_u32(n, lane);
        int at = 0;
        if (lane == 63) at = atomicAdd(count, (int)to);
        uint32_t i = (uint32_t)__builtin_amdgcn_readlane(at, 63) + to - n;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            if ((waiting >> e) & 1) {
                if (i < (uint32_t)LIST) {
                    list[i] = slot[e];
                    slot[e] = i;
                    listed |= 1u << e;
                }
                ++i;
            }
        }
    };
    if (most > kBucketOwn) {                                       // the same in all lanes
#pragma unroll
        for (int e = 0; e < 16; ++e) waiting |= bucket_size(slot[e]) > kBucketOwn ? 1u << e : 0u;
        put();
    }
    __syncthreads();
    const uint32_t some = (uint32_t)count[0];                      // on the list or waiting for it
    for (uint32_t left = some; left != 0;) {
        const uint32_t n = min(left, (uint32_t)LIST), sub = tid & 3;
        left -= n;
        // four lanes to an element, every fourth of its bucket's elements each
#pragma unroll 1
        for (uint32_t i = tid >> 2; i < n; i += T / 4) {
            const uint32_t s = list[i], f = position(s), size = bucket_size(s), r = place(s);
            const uint2 me = kv[f + r];
            uint32_t less = 0;
#pragma unroll 1
            for (uint32_t j = sub; j < size; j += 16) {            // (reads at most fifteen past the bucket)
                static_for<4>([&](auto t) { less = count_below<4 * t>(less, kv[f + j + 4 * t], me, (int)(r - j)); });
            }
            less += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)less, 0xB1, 0xF, 0xF, false);
            less += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)less, 0x4E, 0xF, 0xF, false);
            if (sub == 0) list[i] = f + less;
        }
        __syncthreads();
        const uint32_t now = listed & waiting;
        if (now != 0) {
#pragma unroll
            for (int e = 0; e < 16; ++e)
                if ((now >> e) & 1) slot[e] = list[slot[e]];
        }
        waiting &= ~listed;
        if (left != 0) {
            if (tid == 0) count[0] = 0;                            // (everybody has read it)
            __syncthreads();
            if (__ballot(waiting != 0) != 0ull) put();
            __syncthreads();
        }
    }
    auto rank = [&](auto some_) {
        constexpr bool SOME = decltype(some_)::value;              // is anything on the list?
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            if (SOME && ((listed >> e) & 1)) continue;
            const uint32_t f = position(slot[e]), size = bucket_size(slot[e]), r = place(slot[e]);
            const uint2 me = make_uint2(key[e], __float_as_uint(sv[e]));
            uint32_t less = 0;
            static_for<4>([&](auto t) { less = count_below<t>(less, kv[f + t], me, (int)r); });
            if (most > 4) {
#pragma unroll 1
                for (uint32_t i = 4; i < size; i += 4) {           // (reads at most three past the bucket)
                    static_for<4>([&](auto t) { less = count_below<t>(less, kv[f + i + t], me, (int)(r - i)); });
                }
            }
            slot[e] = f + less;
        }
    };
    if (mine) {
        if (some != 0) rank(std::true_type{});
        else rank(std::false_type{});
    }
    __syncthreads();
    if (mine) {
#pragma unroll
        for (int e = 0; e < 16; ++e) kv[pad16((int)slot[e])] = make_uint2(key[e], __float_as_uint(sv[e]));
    }
    for (int p = K + tid; p < 16 * T; p += T) kv[pad16(p)] = make_uint2(kPadKey, 0u);
    __syncthreads();
    return true;
}

// The least distance of unequal centres, in units of M = max|w_S|, at which the E-step's comparison of two of them is
// monotone along the row whatever the caller's centre_gap.  With distances p, q of a weight to centres d apart and
// u = 2^-53, the rounded squares differ from p^2, q^2 by at most 3 u of them: outside the two centres |p - q| = d, so the
// comparison comes out right where d (p + q) > 3 u (p^2 + q^2), hence for d >= 12 u M; between them both rounded squares
// are monotone in the weight.
constexpr double kLeastGap = 0x1p-49;

template <int BITS, int T>
__global__ __launch_bounds__(T, 4) void quantize_sorted_kernel(
    const float* __restrict__ w, const float* __restrict__ act, const float* __restrict__ u,
    int64_t K64, int symmetric, int iters, double centre_gap, uint8_t* __restrict__ codes_out,
    uint16_t* __restrict__ lut, uint16_t* __restrict__ scale, uint16_t* __restrict__ offset,
    int32_t* __restrict__ msteps) {
    constexpr int L = 1 << BITS;
    constexpr int W = T / kWave;
    constexpr int LOGKP = T == 64 ? 10 : T == 128 ? 11 : T == 256 ? 12 : T == 512 ? 13 : 14;
    static_assert(16 * T == 1 << LOGKP, "16 elements per thread, 1024 to 16384 per block");
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int K = (int)K64, G = K / kGroup;
    uint2* kv = reinterpret_cast<uint2*>(smem);
    float* ws = reinterpret_cast<float*>(smem);
    float* alpha = reinterpret_cast<float*>(smem + sorted_padw(T) * 8);
    double* pre_s = reinterpret_cast<double*>(alpha + T / 8);   // [T + 1]
    double* pre_sx = pre_s + T + 1;             // [T + 1]
    double* scan = pre_sx + T + 1;              // [2 W]
    double* red = pre_s;                        // [W][2][L], per-weight method only: it has no running sums
    double* cen = scan + 2 * W;                 // [L]
    double* cen0 = cen + L;                     // [L]
    uint32_t* fin = reinterpret_cast<uint32_t*>(cen);   // [L] smallest key of the cluster of rank i (none: kPadKey), once cen has been read
    int* misc = reinterpret_cast<int*>(cen0 + L);// [0], [1] selected index (by turns); [2] method flag; [3] .. [6] of the sort ([3] no buckets, [5] length of the list, [6] looks); [4] a weight that is not finite; [40] as below

    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int64_t n = blockIdx.x;
    if (tid == 0) misc[4] = 0;
    scale_row<BITS, T>(w + n * K64, n, G, symmetric, scale, offset, ws, alpha);

    // ---- 2. k-means++ with sample weights; thread t owns the 16 weights from 16 t on, if the row has them, in registers:
    // the scaled weight, the sample weight s and the sampling mass.  The mass is s for the first centre and
    // s * (squared distance to the nearest centre chosen so far) afterwards; as s >= 0, multiplying by s and
    // rounding is monotone, so s * min(d_old, d_new) is min(s * d_old, s * d_new) bit for bit and the
    // distances themselves need not be kept.  Bound: 2^n rounds of five instructions per weight, a third of the time (6144 x 4096: 60 of
    // 180 us), and in every round a chain of sums over the wavefronts, sixteen additions in the thread that holds the draw and two
    // barriers.  (Ten instructions with a comparison and two selects in place of v_min_f64, x converted every time and copies of x and
    // s: 6144 x 4096 any4 588 -> 519 us, 4096 x 14336 1698 -> 1479 us together with the sums of the wavefronts, read several at a time.
    // The sample weights are held in fp64 too: their conversion takes as long as two of the others; 6144 x 4096 493 -> 485 us,
    // 4096 x 14336 1427 -> 1410, no more than runs differ.)
    // Sixteen weights a thread for every K, so that whole wavefronts have none where the row is shorter than the block's
    // 16 T and skip the phases: with the row spread evenly, all of them ran all phases with most lanes idle.  With the
    // codes from the sort's keys (below): 11525 x 1024 any4 726 -> 579 us, 6144 x 4096 528 -> 500, 4096 x 14336 1522 -> 1447.
    const bool mine = tid * 16 < K;                                // (K is a multiple of 128)
    const int j0 = mine ? tid * 16 : 0;
    float xv[16], sv[16];
    {
        bool odd = false;
#pragma unroll
        for (int e = 0; e < 16; ++e) { xv[e] = 0.0f; sv[e] = 0.0f; }
        if (mine) {
            const float a = alpha[j0 >> 7];
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const float4 x4 = reinterpret_cast<const float4*>(ws + j0)[g];
                float4 s4 = make_float4(1.0f, 1.0f, 1.0f, 1.0f);
                if (act) s4 = reinterpret_cast<const float4*>(act + j0)[g];   // (a call's pointers are 16-byte aligned)
                const float x[4] = {x4.x, x4.y, x4.z, x4.w}, s[4] = {s4.x, s4.y, s4.z, s4.w};
#pragma unroll
                for (int i = 0; i < 4; ++i) { xv[4 * g + i] = x[i]; sv[4 * g + i] = a * s[i]; }
            }
#pragma unroll
            for (int e = 0; e < 16; ++e)
                odd |= __builtin_amdgcn_classf(xv[e], 0x207) | __builtin_amdgcn_classf(sv[e], 0x207);   // a NaN or an infinity
        }
        if (odd) misc[4] = 1;
        __syncthreads();
        const bool odd_row = misc[4] != 0;
        // one draw: the threads' masses are summed and scanned, the thread whose chunk holds the draw walks it
        auto draw = [&](int q, double part, auto&& walk) -> double {
            double inc = wave_inclusive_sum(part, lane);
            if (lane == 63) scan[(q & 1) * W + wv] = inc;          // (two sets of partial sums and of the drawn
            if (tid == 0) misc[q & 1] = 0x7FFFFFFF;                // sample, used by turns: one barrier less per centre)
            __syncthreads();
            double base = 0.0, total = 0.0;
#pragma unroll 4
            for (int i = 0; i < W; ++i) {
                base = i == wv ? total : base;
                total += scan[(q & 1) * W + i];
            }
            inc += base;
            double before = wave_shr1_f64(inc);
            if (lane == 0) before = base;
            if (total > 0.0) {
                const double t = (double)u[n * L + q] * total;
                if (mine && before <= t && inc > t) atomicMin(&misc[q & 1], j0 + walk(before, t));
            } else if (tid == 0) {
                const int64_t j = (int64_t)((double)u[n * L + q] * (double)K);
                misc[q & 1] = (int)min(j, (int64_t)K - 1);
            }
            __syncthreads();
            const double cq = (double)ws[min(misc[q & 1], K - 1)];   // (nothing drawn: not reachable with finite, non-negative masses)
            if (tid == 0) { cen[q] = cq; cen0[q] = cq; }
            return cq;
        };
        double mass[16], xd[16], sd[16];
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            sd[e] = (double)sv[e];
            xd[e] = (double)xv[e];
            asm volatile("" : "+v"(xd[e]), "+v"(sd[e]));
            mass[e] = sd[e];
        }
        // With a NaN or an infinity in the row a mass is replaced only by one that compares as smaller: one that is no number
        // from the first centre on stays so, and with it the total (`none`, whatever v_min_f64 makes of the mass); one that
        // would become so later does not.  Rows with a NaN, 6144 x 4096 any4: 1846 -> 857 us against masses computed anew for
        // every centre.
        double none = 0.0;
#pragma unroll 1
        for (int q = 0; q < L; ++q) {
            double part = none;
            if (mine) {
#pragma unroll
                for (int e = 0; e < 16; ++e) part += mass[e];
            }
            const double cq = draw(q, part, [&](double run, double t) -> int {
                // the first weight at which the running mass exceeds t; if rounding leaves none, the last one
                // with any mass
                int pick = 16, last = 0;
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    run += mass[e];
                    last = mass[e] > 0.0 ? e : last;
                    pick = min(pick, run > t ? e : 16);
                    asm volatile("" : "+v"(run), "+v"(pick), "+v"(last));      // (one after the other: sixteen sums at a time hold 32 registers)
                }
                return pick == 16 ? last : pick;
            });
            if (q == 0) {
#pragma unroll
                for (int e = 0; e < 16; ++e) mass[e] = __hiloint2double(0x7FF00000, 0);
                if (odd_row && mine) {
#pragma unroll 1
                    for (int e = 0; e < 16; ++e) {
                        const double d = (double)ws[j0 + e] - cq, m = (double)(alpha[j0 >> 7] * (act ? act[j0 + e] : 1.0f)) * (d * d);
                        none = m != m ? m : none;
                    }
                }
            }
            if (mine) {
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const double d = xd[e] - cq;
                    const double m = sd[e] * (d * d);
                    asm("v_min_f64 %0, %1, %0" : "+v"(mass[e]) : "v"(m));
                    if (e % 4 == 3) __builtin_amdgcn_sched_barrier(0);         // (more of them at a time do not fit the registers)
                }
            }
        }
#pragma unroll
        for (int e = 0; e < 16; ++e) { xv[e] = (float)xd[e]; sv[e] = (float)sd[e]; }        // exact
    }

    // ---- sort the row: elements (order-preserving image of w_S, sample weight), ascending; every thread
    // brings the chunk it holds, and keeps its keys for the codes
    uint32_t key[16];
    {
#pragma unroll
        for (int e = 0; e < 16; ++e) key[e] = f32_key(xv[e]);
        if (!sort_by_buckets<T>(kv, reinterpret_cast<uint32_t*>(scan), reinterpret_cast<uint32_t*>(pre_s), misc + 3, misc + 5,
                                key, sv, mine, K)) {
#pragma unroll
            for (int e = 0; e < 16; ++e)
                kv[tid * 17 + e] = mine ? make_uint2(key[e], __float_as_uint(sv[e])) : make_uint2(kPadKey, 0u);
            __syncthreads();
            sort_first16<T>(kv);
            for (int m = 5; m <= LOGKP; ++m) {
                const int top = m - 1;
                if constexpr (LOGKP > 12) {
                    if (top >= 12) sort_round<T, 12, LOGKP - 12>(kv, m, top);
                }
                if (top >= 8) sort_round<T, 8, LOGKP < 12 ? LOGKP - 8 : 4>(kv, m, min(top, 11));
                if (top >= 4) sort_round<T, 4, 4>(kv, m, min(top, 7));
                sort_round<T, 0, 4>(kv, m, min(top, 3));
            }
        }
    }

    // one sorted element: its scaled weight and sample weight in fp64 (the padding counts as nothing)
    auto element = [&](int p, double& x, double& sw) {
        const uint2 v = kv[pad16(p)];
        const bool real = v.x != kPadKey;
        x = real ? (double)key_f32(v.x) : 0.0;
        sw = real ? (double)__uint_as_float(v.y) : 0.0;
    };

    // ---- running sums of s and s * w_S along the sorted row, one entry per 16 elements
    {
        double cs = 0.0, csx = 0.0;
        int t16 = tid * 16;
        asm volatile("" : "+v"(t16));
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            double x, sw;
            element(t16 + e, x, sw);
            cs += sw;
            csx += sw * x;
        }
        double is = wave_inclusive_sum(cs, lane), isx = wave_inclusive_sum(csx, lane);
        if (lane == 63) { scan[2 * wv] = is; scan[2 * wv + 1] = isx; }
        __syncthreads();
        double bs = 0.0, bsx = 0.0;
#pragma unroll 1
        for (int i = 0; i < wv; ++i) { bs += scan[2 * i]; bsx += scan[2 * i + 1]; }
        is += bs;
        isx += bsx;
        double es = shfl_up_f64(is, 1), esx = shfl_up_f64(isx, 1);
        if (lane == 0) { es = bs; esx = bsx; }
        pre_s[tid] = es;
        pre_sx[tid] = esx;
        if (tid == T - 1) { pre_s[T] = is; pre_sx[T] = isx; }
        __syncthreads();
    }
    // ---- 3, sorted row: the Lloyd passes on wavefront 0.  Lane 16 sub + i holds the centre of rank i (by value, then
    // index): value d, original index own, its range of sorted positions in the last pass.  The four rows of 16 lanes hold
    // the same and split the searches and the sums (sub = 0 .. 3), so a neighbouring centre is a DPP move away.  A pass
    // is one chain of dependent steps, ~20 of them per row of weights, and nothing else of the block runs meanwhile: what
    // counts is its latency.  So a boundary is sought among the first elements of the running sums' chunks, first around
    // where it should have moved to since the last pass (most often the only round of probes), and the one chunk that holds
    // it is read once, for its place in it and for its sums.  4096 x 14336 any4 2070 -> 1698 us, 6144 x 4096 698 -> 588 us
    // against a search of all positions, four neighbouring lanes per centre (a pass of a long row 2.2 -> 1.0 us).
    if (wv == 0) {
        const int i = lane & 15, sub = lane >> 4;
        const bool live = i < L;
        const int nch = K >> 4;                                    // chunks (K is a multiple of 128)
        double d = live ? cen[i] : 0.0;
        int own = i;
        const double maxabs = fmax(fabs((double)key_f32(kv[0].x)), fabs((double)key_f32(kv[pad16(K - 1)].x)));
        const double tol = fmax(centre_gap, kLeastGap) * maxabs;
        const double total_s = pre_s[nch], total_sx = pre_sx[nch];
        int prev_s = -2, prev_e = -2;
        int done = 0, chunk = 0;                                   // chunk: where the centre's lower boundary was last
        float last_mid = 0.0f, density = 0.0f;
        bool fallback = misc[4] != 0, some = false;                // (no order among weights that are no numbers)
        int start = 0;
        auto below_f64 = [](double v) { return row_shr_f64<1>(v); };
        auto below_i32 = [](int v) { return __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, false); };
        auto above_i32 = [](int v) { return __builtin_amdgcn_update_dpp(0, v, 0x101, 0xF, 0xF, false); };
        auto above_f64 = [&](double v) { return __hiloint2double(above_i32(__double2hiint(v)), above_i32(__double2loint(v))); };
        // sum over the four rows of lanes, (row 0 + row 1) + (row 2 + row 3), in every lane
        auto rows_sum = [](double v) {
            const auto h1 = __builtin_amdgcn_permlane16_swap(__double2hiint(v), __double2hiint(v), false, false);
            const auto l1 = __builtin_amdgcn_permlane16_swap(__double2loint(v), __double2loint(v), false, false);
            v = __hiloint2double(h1[0], l1[0]) + __hiloint2double(h1[1], l1[1]);
            const auto h2 = __builtin_amdgcn_permlane32_swap(__double2hiint(v), __double2hiint(v), false, false);
            const auto l2 = __builtin_amdgcn_permlane32_swap(__double2loint(v), __double2loint(v), false, false);
            return __hiloint2double(h2[0], l2[0]) + __hiloint2double(h2[1], l2[1]);
        };
        // how many of a centre's four lanes say yes
        auto count4 = [&](bool b) -> int {
            const unsigned long long m = __ballot(b) >> i;
            return __popc((unsigned)m & 0x00010001u) + __popc((unsigned)(m >> 32) & 0x00010001u);
        };
        while (!fallback) {
            // the centres in order of (value, index)?  Ranked anew, 2^n comparisons per centre, only where they are not
            // (the centres of a one-dimensional k-means hardly ever overtake each other)
            double dprev = below_f64(d);
            int own_prev = below_i32(own);
            if (__ballot(live && i > 0 && !(dprev < d || (dprev == d && own_prev < own))) != 0ull) {
                int r = 0;
                static_for<L>([&](auto p_) {
                    constexpr int p = decltype(p_)::value;
                    const double dp = lane_f64<p>(d);
                    const int op = __builtin_amdgcn_readlane(own, p);
                    r += (dp < d || (dp == d && op < own)) ? 1 : 0;
                });
                const int to = ((lane & 48) | (live ? r : i)) * 4;   // the ranks are a permutation of the live centres
                d = __hiloint2double(__builtin_amdgcn_ds_permute(to, __double2hiint(d)),
                                     __builtin_amdgcn_ds_permute(to, __double2loint(d)));
                own = __builtin_amdgcn_ds_permute(to, own);
                prev_s = __builtin_amdgcn_ds_permute(to, prev_s);
                prev_e = __builtin_amdgcn_ds_permute(to, prev_e);
                dprev = below_f64(d);
                own_prev = below_i32(own);
            }
            // equal centres: only the lowest index ever wins a weight; it stands for the run
            const bool rep = live && (i == 0 || dprev != d);
            const unsigned repmask = (unsigned)__ballot(rep) & 0xFFFFu;
            const bool distinct = repmask == (1u << L) - 1u;
            const unsigned above = repmask & ~((2u << i) - 1u);
            const int nxt = above ? __ffs((int)above) - 1 : -1;    // the next run's centre
            int a_own = own_prev;                                  // index of the run below
            if (!distinct) {
                const unsigned below = repmask & ((1u << i) - 1u);
                a_own = __shfl(own, below ? 31 - __clz((int)below) : 0);
            }
            const bool seek = rep && i > 0;
            bool bad = seek && (d - dprev) <= tol;
            // the E-step's own comparison: does this centre win x from the one below it?  False up to some position
            // of the sorted row and true from there on.
            auto wins = [&](double x) {
                const double da = x - dprev, db = x - d;
                const double dda = da * da, ddb = db * db;
                return (ddb < dda) | ((ddb == dda) & (own < a_own));   // (no branches: they cost more than the comparison)
            };
            auto first_of = [&](int c) { return (double)key_f32(kv[c * 17].x); };
            // lo = the number of chunks whose first element it does not win, in [lo, hi]; a round probes four of them
            int lo = 0, hi = seek ? nch : 0;
            const float mid = 0.5f * (float)(dprev + d);
            if (done > 0) {                                        // where it should be, as it moved by mid - last_mid
                const int guess = chunk + (int)rintf(fminf(fmaxf((mid - last_mid) * density, -16384.0f), 16384.0f));
                auto at = [&](int k) { return min(max(guess - 1 + k, 0), nch - 1); };
                const int losses = count4(!wins(first_of(at(sub))));
                if (seek) {
                    if (losses > 0) lo = at(losses - 1) + 1;
                    if (losses < 4) hi = at(losses);
                }
            }
            while (__ballot(lo < hi) != 0ull) {                    // the inner fifths of the open range
                const int span = hi - lo;
                const int probe = lo + (span * (sub + 1)) / 5;     // lo <= probe < hi while the range is open
                const int losses = count4(!wins(first_of(min(probe, nch - 1))));
                if (lo < hi) {
                    const int lo2 = losses > 0 ? lo + (span * losses) / 5 + 1 : lo;
                    const int hi2 = losses < 4 ? lo + (span * (losses + 1)) / 5 : hi;
                    lo = lo2;
                    hi = hi2;
                }
            }
            chunk = min(max(lo - 1, 0), nch - 1);
            // its place in the chunk, and the running sums before it: four elements per lane
            double ss = 0.0, sx = 0.0;
            int before = 0;
            uint2 v[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) v[k] = kv[chunk * 17 + sub + 4 * k];
            const int c0 = max(chunk - 2, 0), c1 = min(chunk + 2, nch - 1);
            const uint32_t key0 = kv[c0 * 17].x, key1 = kv[c1 * 17].x;
            const double run_s = pre_s[chunk], run_sx = pre_sx[chunk];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const double x = (double)key_f32(v[k].x), sw = (double)__uint_as_float(v[k].y);
                const bool lose = seek & !wins(x);
                const double sw0 = lose ? sw : 0.0, sx0 = lose ? sw * x : 0.0;
                ss += sw0;
                sx += sx0;
                before += count4(lose);
            }
            start = seek ? chunk * 16 + before : 0;
            ss = rows_sum(ss) + run_s;
            sx = rows_sum(sx) + run_sx;
            // (the row's end takes the running sums' own entry: the mass of an empty last cluster is exactly 0)
            ss = start == K ? total_s : ss;
            sx = start == K ? total_sx : sx;
            last_mid = mid;                                        // chunks per unit of weight around it, for the next guess
            density = (float)(c1 - c0) * __builtin_amdgcn_rcpf(key_f32(key1) - key_f32(key0));
            // the range ends where the next run's begins
            int s_nxt = above_i32(start);
            double e_ss = above_f64(ss), e_sx = above_f64(sx);
            if (!distinct) {
                s_nxt = __shfl(start, max(nxt, 0));
                e_ss = shfl_f64(ss, max(nxt, 0));
                e_sx = shfl_f64(sx, max(nxt, 0));
            }
            const int end = nxt < 0 ? K : s_nxt;
            bad = bad || (rep && end < start);
            const double den = (nxt < 0 ? total_s : e_ss) - ss;
            const double num = (nxt < 0 ? total_sx : e_sx) - sx;
            // did any weight change its centre?  compare every centre's range with the previous pass
            some = rep && start < end;
            const int rs = some ? start : -1, re = some ? end : -1;
            const bool changed = __ballot(live && (rs != prev_s || re != prev_e)) != 0ull;
            if (__ballot(bad) != 0ull) { fallback = true; break; }
            if ((done > 0 && !changed) || done >= iters) break;
            prev_s = rs;
            prev_e = re;
            if (rep && den > 0.0) d = num / den;                   // M-step, Eq. (B); no weight: the centre stays
            ++done;
        }
        if (lane == 0) misc[2] = fallback ? 1 : 0;
        if (!fallback) {
            // ---- 4. the centre of rank i: table entry i, and code i for every weight from the first of its range up to
            // the first of the next non-empty range
            if (live && sub == 0) {
                lut[n * L + i] = (uint16_t)f32_to_bf16((float)d);
                fin[i] = some ? kv[pad16(start)].x : kPadKey;
            }
            if (msteps && lane == 0) msteps[n] = done;
        }
    }
    __syncthreads();
    if (misc[2] != 0) {
        // two unequal centres too close for the sorted search, or a weight that is not finite: the row again, per weight, from its starting centres
        __syncthreads();
        scale_row<BITS, T>(w + n * K64, n, G, symmetric, scale, offset, ws, alpha);
        if (tid < L) cen[tid] = cen0[tid];
        __syncthreads();
        lloyd_per_weight_lean<BITS, T>(ws, smem + (size_t)K * 4, alpha, red, cen, misc, act, K, iters, n, codes_out, lut,
                                       msteps);
        return;
    }
    // the codes in row order: every weight's place among the clusters' smallest members; a cluster never splits equal
    // weights, so this is its range.  The smallest members ascend with the rank once an empty cluster takes that of the next
    // one, so four comparisons and the selects of what to compare with do (15 comparisons and selects otherwise).  The keys
    // are those of the sort: scaling the row once more cost a read and a division per weight.
    if (mine) {
        uint32_t fk[L];
        fk[L - 1] = fin[L - 1];
#pragma unroll
        for (int i = L - 2; i > 0; --i) fk[i] = min(fin[i], fk[i + 1]);
        uint32_t out[4] = {};
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            uint32_t f[L], code = 0;                               // f[i]: fk[i] among those still in question
#pragma unroll
            for (int i = 1; i < L; ++i) f[i] = fk[i];
#pragma unroll
            for (int h = L / 2; h > 0; h >>= 1) {
                const bool up = key[e] >= f[h];
                code |= up ? (uint32_t)h << (8 * (e & 3)) : 0u;
#pragma unroll
                for (int i = 1; i < h; ++i) f[i] = up ? f[h + i] : f[i];
            }
            out[e >> 2] |= code;
        }
        *reinterpret_cast<uint4*>(codes_out + n * K64 + j0) = make_uint4(out[0], out[1], out[2], out[3]);
    }
}

size_t quantize_max_k() {
    // the row, its codes and the scratch have to fit the 160 KB of LDS of one compute unit
    return 28672;
}

hipError_t launch_quantize(const float* w, const float* act, const float* u, int64_t N, int64_t K, int bits,
                           int symmetric, int iters, double centre_gap, uint8_t* codes, uint16_t* lut, uint16_t* scale,
                           uint16_t* offset, int32_t* msteps, hipStream_t stream) {
    if (N > 0x7FFFFFFF || K > (int64_t)quantize_max_k()) return hipErrorInvalidValue;
    hipError_t e = hipSuccess;
    if (centre_gap >= 0.0 && K <= kSortedMaxK) {
#define ANY4_QUANT_S(B, T)                                                                                        \
    do {                                                                                                          \
        e = ensure_lds<quantize_sorted_kernel<B, T>>((int)sorted_lds_bytes(T, B));                                \
        if (e != hipSuccess) return e;                                                                            \
        hipLaunchKernelGGL((quantize_sorted_kernel<B, T>), dim3((unsigned)N), dim3(T), sorted_lds_bytes(T, B), stream, w, \
                           act, u, K, symmetric, iters, centre_gap, codes, lut, scale, offset, msteps);           \
    } while (0)
        // The smallest block that holds the row: a compute unit holds 16 wavefronts of this kernel, so a row of at most 1024
        // weights in a block of one wavefront has 15 others beside it and in one of four only three.  any4 against four
        // wavefronts, when these were measured: 11525 x 1024 584 -> 270 us, 11525 x 1152 645 -> 411 us, 28000 x 2048 1650 ->
        // 1074 us; 512 x 1024, where the chip is nearly empty either way, 57 us both.
#define ANY4_QUANT_ST(B)                                                                                          \
    do {                                                                                                          \
        if (K <= 1024) ANY4_QUANT_S(B, 64);                                                                       \
        else if (K <= 2048) ANY4_QUANT_S(B, 128);                                                                 \
        else if (K <= 4096) ANY4_QUANT_S(B, 256);                                                                 \
        else if (K <= 8192) ANY4_QUANT_S(B, 512);                                                                 \
        else ANY4_QUANT_S(B, 1024);                                                                               \
    } while (0)
        switch (bits) {
            case 4: ANY4_QUANT_ST(4); break;
            case 3: ANY4_QUANT_ST(3); break;
            default: ANY4_QUANT_ST(2); break;
        }
#undef ANY4_QUANT_ST
#undef ANY4_QUANT_S
        return hipGetLastError();
    }
    const size_t lds = quantize_lds_bytes(K, bits);
#define ANY4_QUANT(B)                                                                                             \
    do {                                                                                                          \
        e = ensure_lds<quantize_kernel<B>>((int)quantize_lds_bytes((int64_t)quantize_max_k(), B));                \
        if (e != hipSuccess) return e;                                                                            \
        hipLaunchKernelGGL(quantize_kernel<B>, dim3((unsigned)N), dim3(QT), lds, stream, w, act, u, K, symmetric, \
                           iters, codes, lut, scale, offset, msteps);                                             \
    } while (0)
    switch (bits) {
        case 4: ANY4_QUANT(4); break;
        case 3: ANY4_QUANT(3); break;
        default: ANY4_QUANT(2); break;
    }
#undef ANY4_QUANT
    return hipGetLastError();
}

}  // namespace any4
