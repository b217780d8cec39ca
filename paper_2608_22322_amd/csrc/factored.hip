// Factored-state optimizer steps on gfx950: Adafactor (factored second
// moment) and CAME (factored second moment + factored confidence + dense
// momentum), section 3.1, with AL/UF8/FP32 codes per state role (section 4).
//
// Kernel sequence of one Adafactor step (2-D tensors):
//   marg   row and column partial sums of g^2 per unit, with a bounded error;
//          its leading workgroups run the whole step of the 1-D tensors
//   mean   per 64 elements of R or C: the unit partials merged, eps1 added to
//          the mean, EMA rounded to fp32, sums for mean(R)
//   enc    per code block of R and C: re-encoded, and the factors
//          r_i = (R_i / mean R)^-1/2, c_j = C_j^-1/2
//   rms    partial sums of u^2, u_ij = (r_i c_j) g_ij, per unit
//   clip   per tensor: max(1, RMS(u) / d)
//   apply  p <- p (1 - lr wd) - lr u / clip
// CAME adds: res (sums of (uhat - m)^2 + eps2 with the in-step momentum),
// mean and enc over the confidence, and apply (recompute uhat and m, encode m, update p).
//
// Marginal sums. The matrices are cut into units of a.ur rows x 256 columns
// (ur = 256 for large lists, fewer rows for lists that would leave the chip
// idle), one wavefront per unit. Every partial is one binary64 sum with a
// proven relative error bound (below); the finalize step keeps the fast sum
// only where that cannot change the fp32 rounding of the state's EMA and
// otherwise sums the element's row or column again exactly, so the fp32 states
// (and their codes) are the ones of the exactly rounded means.
#include "al_device.hpp"
#include "al_internal.hpp"

namespace al {

// ------------------------------------------------------------------ helpers
// Global-address-space view of the data pointers of a descriptor (the
// descriptors are read from the workspace, so their pointers are generic to
// the compiler; see gp in al_device.hpp).
struct GD {
    gp<float> p;
    gp<const void> g;
    gp<void> m;
    gp<float> mm;
    gp<double> colpart, rowpart;
    gp<const double> rfac, cfac, sr, sc;
    gp<const double> scal;
    int64_t rows, cols, unit_begin, ach_begin;
    int32_t nru, ncu;
};

__device__ __forceinline__ GD gview(const FacDesc& d) {
    GD v;
    v.p = to_g(d.p);
    v.g = to_g(d.g);
    v.m = to_g(d.m);
    v.mm = to_g(d.mm);
    v.colpart = to_g(d.colpart);
    v.rowpart = to_g(d.rowpart);
    v.rfac = to_g((const double*)d.rfac);
    v.cfac = to_g((const double*)d.cfac);
    v.sr = to_g((const double*)d.sr);
    v.sc = to_g((const double*)d.sc);
    v.scal = to_g((const double*)d.scal);
    v.rows = d.rows;
    v.cols = d.cols;
    v.unit_begin = d.unit_begin;
    v.ach_begin = d.ach_begin;
    v.nru = d.nru;
    v.ncu = d.ncu;
    return v;
}

// Term of the second moment's marginal sums: fl64(g^2 + eps1).
__device__ __forceinline__ double marg_term(float g, double eps1) {
    const double x = (double)g;
    return x * x + eps1;
}

// Term of CAME's confidence marginal sums, from the decoded momentum and the
// clipped update: m = fl32(beta1 mhat + (1 - beta1) uhat), (uhat - m)^2 + eps2.
__device__ __forceinline__ double res_term(const FacArgs& a, float mh, float uh) {
    const float m = (float)(a.beta1 * (double)mh + a.omb1 * (double)uh);
    const double df = (double)uh - (double)m;
    return df * df + a.eps2;
}

// uhat - m of the same term (exact in binary64): the whole-unit residual pass
// accumulates its square with fused multiply-adds and adds eps2 to the mean.
__device__ __forceinline__ double res_diff(const FacArgs& a, float mh, float uh) {
    const float m = (float)(a.beta1 * (double)mh + a.omb1 * (double)uh);
    return (double)uh - (double)m;
}

// Decode element i of a vector state (runtime codec / block).
__device__ __forceinline__ float vec_decode(int codec, int B, const void* codes, const float* meta, int64_t i,
                                            const Exp2Coef& cf) {
    if (codec == FP32) return reinterpret_cast<const float*>(codes)[i];
    if (codec == UF8) {
        const int32_t q = reinterpret_cast<const int8_t*>(codes)[i];
        return uf8_decode(q, div127((double)meta[i / B]));
    }
    const uint32_t q = codec == AL16 ? reinterpret_cast<const uint16_t*>(codes)[i]
                                     : reinterpret_cast<const uint8_t*>(codes)[i];
    if (q == 0u) return 0.0f;
    const int64_t b = i / B;
    const double step = (double)meta[2 * b + 1] / (codec == AL16 ? 65534.0 : 254.0);
    return al_decode_fast(q, (double)meta[2 * b], step, cf);
}

// Encode x[0, n) into a vector state, one block per wavefront at a time
// (runtime codec / block; the vectors are small). Padding codes are 0.
__device__ void vec_encode(int codec, int B, const float* x, int64_t n, float log_floor, void* codes, float* meta,
                           int wave, int nwaves, int lane) {
    if (codec == FP32) {
        for (int64_t i = (int64_t)wave * 64 + lane; i < n; i += (int64_t)nwaves * 64)
            reinterpret_cast<float*>(codes)[i] = x[i];
        return;
    }
    const int64_t nb = (n + B - 1) / B;
    for (int64_t b = wave; b < nb; b += nwaves) {
        const int64_t s = b * B;
        const int64_t e = s + B < n ? s + B : n;
        if (codec == UF8) {
            uint32_t am = 0u;
            for (int64_t i = s + lane; i < e; i += 64) am = OpMax::f(am, abs_bits(x[i]));
            am = group_reduce<OpMax, 64>(am);
            const double r = am != 0u ? rdiv127((double)u2f(am)) : 0.0;
            if (lane == 0) meta[b] = u2f(am);
            for (int64_t i = s + lane; i < s + B; i += 64) {
                const int32_t q = i < e ? (int32_t)__builtin_rint((double)x[i] * r) : 0;
                reinterpret_cast<int8_t*>(codes)[i] = (int8_t)q;
            }
        } else {
            uint32_t mn = 0xFFFFFFFFu, mx = 0u;
            for (int64_t i = s + lane; i < e; i += 64) {
                mn = OpMin::f(mn, pos_min_key(x[i]));
                mx = OpMax::f(mx, pos_max_key(x[i]));
            }
            mn = group_reduce<OpMin, 64>(mn);
            mx = group_reduce<OpMax, 64>(mx);
            const ALFit f = al_fit(mn, mx, log_floor);
            if (lane == 0) {
                meta[2 * b] = f.any ? (float)f.lmin : 0.0f;
                meta[2 * b + 1] = f.any ? (float)f.delta : 0.0f;
            }
            const int levels = codec == AL16 ? 65534 : 254;
            const ALEnc enc = al_enc_params(f.lmin, f.any ? (double)levels / f.delta : 1.0);
            for (int64_t i = s + lane; i < s + B; i += 64) {
                const float v = i < e ? x[i] : 0.0f;
                const uint32_t q = codec == AL16 ? al_encode_fast<65534>(v, enc) : al_encode_fast<254>(v, enc);
                if (codec == AL16)
                    reinterpret_cast<uint16_t*>(codes)[i] = (uint16_t)q;
                else
                    reinterpret_cast<uint8_t*>(codes)[i] = (uint8_t)q;
            }
        }
    }
}

// Block-wide (256 threads) double-double total in a fixed order.
__device__ DD block_dd_sum(DD v, DD* sh) {
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    v = dd_wave_sum(v);
    if (lane == 0) sh[w] = v;
    __syncthreads();
    DD t = sh[0];
    for (int k = 1; k < (int)(blockDim.x >> 6); ++k) t = dd_merge(t, sh[k]);
    __syncthreads();
    return t;
}

// --------------------------------------------------------------- descriptors
// The packed first units / chunks / tiles / blocks (kFacIndex arrays of nt) go
// behind the table, for the searches.
__global__ __launch_bounds__(64) void fac_desc_copy_kernel(const FacRecBatch b, int count, int first, int words, char* ws,
                                                           size_t index_off, int nt, int ur) {
    const int k = threadIdx.x;
    if (k >= count) return;
    const uint64_t* const r = b.w + k * words;
    const bool came = words > kFacRecAda;
    FacDesc d;
    d.p = reinterpret_cast<float*>(r[kRecP]);
    d.g = reinterpret_cast<const void*>(r[kRecG]);
    d.rows = (int64_t)r[kRecRows];
    d.cols = (int64_t)r[kRecCols];
    const bool fac = d.rows > 1;
    void* const s0 = reinterpret_cast<void*>(r[kRecS0]);
    float* const s1 = reinterpret_cast<float*>(r[kRecS1]);
    d.v = fac ? nullptr : s0;
    d.vm = fac ? nullptr : s1;
    d.vr = fac ? s0 : nullptr;
    d.vrm = fac ? s1 : nullptr;
    d.vc = reinterpret_cast<void*>(r[kRecS2]);
    d.vcm = reinterpret_cast<float*>(r[kRecS3]);
    d.m = came ? reinterpret_cast<void*>(r[kRecM]) : nullptr;
    d.mm = came ? reinterpret_cast<float*>(r[kRecMm]) : nullptr;
    d.cr = came ? reinterpret_cast<void*>(r[kRecCr]) : nullptr;
    d.crm = came ? reinterpret_cast<float*>(r[kRecCrm]) : nullptr;
    d.cc = came ? reinterpret_cast<void*>(r[kRecCc]) : nullptr;
    d.ccm = came ? reinterpret_cast<float*>(r[kRecCcm]) : nullptr;
    d.unit_begin = (int64_t)r[kRecUnit];
    d.ach_begin = (int64_t)r[kRecAch];
    d.mt_begin = (int64_t)r[kRecMt];
    d.blk_begin[0] = (int64_t)r[kRecBlk0];
    d.blk_begin[1] = (int64_t)r[kRecBlk1];
    fac_regions(d, ws, r[kRecOff], came, ur);
    reinterpret_cast<FacDesc*>(ws)[first + k] = d;
    int64_t* const x = reinterpret_cast<int64_t*>(ws + index_off) + first + k;
    x[0] = d.unit_begin;
    x[nt] = d.ach_begin;
    x[2 * nt] = d.mt_begin;
    x[3 * nt] = d.blk_begin[0];
    x[4 * nt] = d.blk_begin[1];
}

hipError_t fac_copy_desc(const FacRec* host, int count, char* ws, size_t index_off, bool came, int ur, hipStream_t s) {
    const int words = came ? (int)kFacRecWords : (int)kFacRecAda;
    const int per = kFacBatchWords / words;
    static_assert(kFacBatchWords / kFacRecAda <= 64, "one thread per record");
    static_assert(sizeof(FacRecBatch) + 64 <= 4096, "copy arguments");
    for (int off = 0; off < count; off += per) {
        FacRecBatch b;
        const int nb = count - off < per ? count - off : per;
        for (int i = 0; i < nb; ++i)
            for (int w = 0; w < words; ++w) b.w[i * words + w] = host[off + i].w[w];
        hipLaunchKernelGGL(fac_desc_copy_kernel, dim3(1), dim3(64), 0, s, b, nb, off, words, ws, index_off, count, ur);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// One wavefront per unit (4 per 256-thread workgroup); lists beyond 2^33 units
// take several launches.
template <class K>
static hipError_t launch_wave_per_unit(K kernel, const FacArgs& a, hipStream_t s) {
    constexpr int64_t kMaxGrid = int64_t(1) << 31;
    for (int64_t base = 0; base < a.total_units; base += 4 * kMaxGrid) {
        const int64_t left = (a.total_units - base + 3) / 4;
        const int64_t grid = left < kMaxGrid ? left : kMaxGrid;
        hipLaunchKernelGGL(kernel, dim3((unsigned)grid), dim3(256), 0, s, a, base);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// ------------------------------ marginal sums over whole units (streaming)
// Units of 256 x 256 in matrices whose width is a multiple of 256: no guards,
// and every unit row starts 16-byte aligned. A batch is P::NR unit rows.
// Lane l = 32 h + q reads columns 8q .. 8q + 7 of rows 2k + h of the
// batch: 16 bytes of bf16 gradients per lane, one load instruction per pair of
// unit rows, later batches' loads issued before the current batch's
// arithmetic. Both sums take the terms as squares t^2 by fused multiply-adds
// (g^2 for the second moment, (uhat - m)^2 for CAME's residual; one rounding
// per term, u = 2^-53); the additive eps1 / eps2 joins the mean in the
// finalize. Rows: a lane's 8 terms (<= 8u) are staged in LDS, and 4 or 8 lanes
// finish each row pairwise and by DPP (<= 5u more): <= 13u. Columns of the
// second moment: plain runs over 16 of the lane's rows, the 8 runs of the unit
// added, the even- and odd-row halves merged (<= 25u); CAME's residual: one
// plain sum over the lane's 128 rows and the merge (<= 129u). The oracle's
// terms fl64(fl64(t^2) + eps) are within 2u of t^2 + eps. The finalize step's
// robustness margin covers these bounds.
constexpr int kWStride = 34;  // LDS stride of a staged row, in doubles (16-byte aligned rows)
constexpr int kWRunRows = 32; // unit rows per plain column run (16 rows of each lane)

template <int G>
struct Raw8 {
    uint4 w;  // 8 bf16
};
template <>
struct Raw8<G_F32> {
    float4 a, b;
};

template <int G>
__device__ __forceinline__ void unpack8(const Raw8<G>& r, float gv[8]) {
    if constexpr (G == G_BF16) {
        const uint32_t w[4] = {r.w.x, r.w.y, r.w.z, r.w.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            gv[2 * i] = u2f(w[i] << 16);
            gv[2 * i + 1] = u2f(w[i] & 0xFFFF0000u);
        }
    } else {
        gv[0] = r.a.x, gv[1] = r.a.y, gv[2] = r.a.z, gv[3] = r.a.w;
        gv[4] = r.b.x, gv[5] = r.b.y, gv[6] = r.b.z, gv[7] = r.b.w;
    }
}

__device__ __forceinline__ double sum8(const double t[8]) {
    return ((t[0] + t[1]) + (t[2] + t[3])) + ((t[4] + t[5]) + (t[6] + t[7]));
}

// Gradients of a batch of NR unit rows (NR / 2 row pairs) of one lane.
template <int G, int NR>
struct WBatch {
    Raw8<G> r[NR / 2];
};

// Batch at unit row rb: the wave-uniform part of each address (row base) plus
// the lane's 32-bit offset lo, so the loads take the scalar-base form.
template <int G, int NR>
__device__ __forceinline__ void load_wbatch(WBatch<G, NR>& b, gp<const void> g, int64_t rb, int64_t cols, uint32_t lo) {
#pragma unroll
    for (int k = 0; k < NR / 2; ++k) {
        if constexpr (G == G_BF16) {
            const gp<const uint16_t> row = g_as<const uint16_t>(g) + (rb + 2 * k) * cols;
            b.r[k].w = ld_u4<false>(g_as<const void>(row + lo));
        } else {
            const gp<const float> row = g_as<const float>(g) + (rb + 2 * k) * cols;
            b.r[k].a = ld_f4<false>(row + lo);
            b.r[k].b = ld_f4<false>(row + lo + 4);
        }
    }
}

// Shared part of the whole-unit marginal kernels, batches of P::NR unit rows
// (4, 8 or 16). The policy P supplies the batch type, load(batch, rb) for the
// rows from rb, and terms(batch, k, t): 8 binary64 values of the lane's row
// 2k + h of that batch whose squares are the terms; P::DEPTH batches are in
// flight (2: the next batch's loads are issued before the current batch's
// arithmetic; 3: the next two). Row partials go to rowpart, column partials to
// colpart, one binary64 sum each; stage holds 2 P::FR x kWStride doubles.
template <class P>
__device__ __forceinline__ void whole_unit_sums(const P& pol, const GD& d, int64_t ru, int64_t cu, double* stage) {
    // row partials are finished P::FR rows (FB batches) at a time
    constexpr int NR = P::NR, NP = NR / 2, FR = P::FR, FB = FR / NR;
    constexpr int LPR = 64 / FR, PPL = 32 / LPR;  // lanes per finished row, partials per lane
    constexpr int SZ = FR * kWStride;  // one stage buffer; finish groups alternate between two
    static_assert(NR == 4 || NR == 8 || NR == 16, "batch rows");
    static_assert(FR % NR == 0 && (FR == 4 || FR == 8 || FR == 16), "finish group rows");
    const int lane = threadIdx.x & 63, h = lane >> 5, q = lane & 31;
    const int64_t r0 = ru * 256, c0 = cu * 256, cols = d.cols;
    const int rrow = lane / LPR, rpart = lane % LPR;  // row finishing: row rrow of a group, partials PPL rpart ..
    // column sums: runs in crun added into cacc (all terms of a batch at once), else one plain sum in cacc
    double cacc[8], crun[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        cacc[j] = 0.0;
        crun[j] = 0.0;
    }
    // Row rrow of finish group gi from its staged partials PPL rpart .. PPL rpart + PPL - 1, pairwise,
    // then merged over the row's LPR lanes. Called one batch late (with the next group's first batch),
    // so the LDS round trip overlaps that batch's arithmetic.
    auto finish_rows = [&](int gi) {
        const double* st = stage + (gi & 1) * SZ + rrow * kWStride + PPL * rpart;
        double rs;
        const double2 p0 = *reinterpret_cast<const double2*>(st);
        if constexpr (PPL == 8) {
            const double2 p1 = *reinterpret_cast<const double2*>(st + 2);
            const double2 p2 = *reinterpret_cast<const double2*>(st + 4);
            const double2 p3 = *reinterpret_cast<const double2*>(st + 6);
            rs = ((p0.x + p0.y) + (p1.x + p1.y)) + ((p2.x + p2.y) + (p3.x + p3.y));
        } else if constexpr (PPL == 4) {
            const double2 p1 = *reinterpret_cast<const double2*>(st + 2);
            rs = (p0.x + p0.y) + (p1.x + p1.y);
        } else {
            rs = p0.x + p0.y;
        }
        rs += dpp_d<kDppQuadXor1>(rs);
        rs += dpp_d<kDppQuadXor2>(rs);
        if constexpr (LPR >= 8) rs += dpp_d<kDppRowHalfMirror>(rs);
        if constexpr (LPR == 16) rs += dpp_d<kDppRowMirror>(rs);
        if (rpart == 0) d.rowpart[cu * d.rows + r0 + FR * gi + rrow] = rs;
    };
    typename P::Batch A, B;
    pol.load(A, 0);
    auto step = [&](const typename P::Batch& cur, int bi) {
        double* sb = stage + ((bi / FB) & 1) * SZ + (bi % FB) * NR * kWStride;
        if constexpr (P::ILP) {
            // all terms of the batch at once (more registers, fewer waves per SIMD, more independent
            // work per wave): the batch's column terms are added first, then into the run
            double cs[8];
#pragma unroll
            for (int k = 0; k < NP; ++k) {
                double t[8];
                pol.terms(cur, k, t);
                double rs = t[0] * t[0];
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    cs[j] = k == 0 ? t[j] * t[j] : __builtin_fma(t[j], t[j], cs[j]);
                    if (j > 0) rs = __builtin_fma(t[j], t[j], rs);
                }
                sb[(2 * k + h) * kWStride + q] = rs;
            }
#pragma unroll
            for (int j = 0; j < 8; ++j) crun[j] += cs[j];
        } else {
            // column sums and the lane's row partial take the squares by fused multiply-adds (one
            // rounding per term)
#pragma unroll
            for (int k = 0; k < NP; ++k) {
                double t[8];
                pol.terms(cur, k, t);
                double rs = t[0] * t[0];
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    cacc[j] = __builtin_fma(t[j], t[j], cacc[j]);
                    if (j > 0) rs = __builtin_fma(t[j], t[j], rs);
                    // two row pairs' terms live at a time: without the fence the compiler forms all terms
                    // of the batch before the column additions
                    if (k & 1) __asm__ volatile("" : "+v"(cacc[j]));
                }
                sb[(2 * k + h) * kWStride + q] = rs;
            }
        }
        // the stages belong to this wavefront alone and its LDS accesses
        // execute in order: only the compiler must keep them in order
        __builtin_amdgcn_wave_barrier();
        if (bi > 0 && bi % FB == 0) finish_rows(bi / FB - 1);
        __builtin_amdgcn_wave_barrier();
        if (P::ILP && (bi + 1) % (kWRunRows / NR) == 0) {
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                cacc[j] += crun[j];
                crun[j] = 0.0;
            }
        }
    };
    // The last pair of batches is peeled: with a conditional load inside the
    // loop the compiler's wait counts would have to hold for both paths, and
    // every odd batch would wait for the next even batch's loads.
    constexpr int NB = 256 / NR;
    if constexpr (P::DEPTH == 2) {
#pragma unroll 1
        for (int bi = 0; bi < NB - 2; bi += 2) {
            pol.load(B, (bi + 1) * NR);
            step(A, bi);
            pol.load(A, (bi + 2) * NR);
            step(B, bi + 1);
        }
        pol.load(B, (NB - 1) * NR);
        step(A, NB - 2);
        step(B, NB - 1);
    } else {
        // three batches rotate, two in flight ahead of the one being formed
        static_assert(P::DEPTH == 3 && NB % 3 == 1, "three-deep rotation over NB = 1 mod 3 batches");
        typename P::Batch C;
        pol.load(B, NR);
#pragma unroll 1
        for (int bi = 0; bi < NB - 4; bi += 3) {
            pol.load(C, (bi + 2) * NR);
            step(A, bi);
            pol.load(A, (bi + 3) * NR);
            step(B, bi + 1);
            pol.load(B, (bi + 4) * NR);
            step(C, bi + 2);
        }
        pol.load(C, (NB - 2) * NR);
        step(A, NB - 4);
        pol.load(A, (NB - 1) * NR);
        step(B, NB - 3);
        step(C, NB - 2);
        step(A, NB - 1);
    }
    __builtin_amdgcn_wave_barrier();
    finish_rows(NB / FB - 1);
    // the two halves hold the even and the odd rows of the same columns
#pragma unroll
    for (int j = 0; j < 8; ++j) cacc[j] += __shfl_xor(cacc[j], 32);
    // through LDS, so that each store instruction writes 64 consecutive
    // column partials (512 bytes) instead of 8 bytes in every 64
    static_assert(2 * SZ >= 256, "the stages hold a unit's 256 column sums");
    __builtin_amdgcn_wave_barrier();
    if (h == 0) {
#pragma unroll
        for (int j = 0; j < 8; ++j) stage[8 * q + j] = cacc[j];
    }
    __builtin_amdgcn_wave_barrier();
    const gp<double> cp = d.colpart + (ru * cols + c0 + lane);
#pragma unroll
    for (int i = 0; i < 4; ++i) cp[64 * i] = stage[lane + 64 * i];
}

// The lane's place in a whole unit: the unit's first gradient element as a
// wave-uniform byte address and the lane's element offset from it.
struct WholeLane {
    int64_t r0, c0, cols;
    uint32_t lo;  // h * cols + 8 q
    int h, q;
};

__device__ __forceinline__ WholeLane whole_lane(const GD& d, int64_t ru, int64_t cu) {
    WholeLane w;
    w.h = (int)(threadIdx.x >> 5) & 1;
    w.q = (int)threadIdx.x & 31;
    w.r0 = ru * 256;
    w.c0 = cu * 256;
    w.cols = d.cols;
    w.lo = (uint32_t)(w.h * d.cols + 8 * w.q);
    return w;
}

template <int G>
__device__ __forceinline__ gp<const void> unit_base(const GD& d, const WholeLane& w) {
    return g_as<const void>(g_as<const uint8_t>(d.g) + (G == G_BF16 ? 2 : 4) * (w.r0 * w.cols + w.c0));
}

// Terms of the second moment's marginals: g^2 (exact in binary64).
template <int G>
struct MargTerms {
    // 8-row batches, all terms of a batch at once: the cheap terms gain more from independent work per
    // wave than from occupancy (2 waves per SIMD)
    static constexpr int NR = 8;
    static constexpr int FR = NR;
    static constexpr bool ILP = true;
    static constexpr int DEPTH = 2;
    using Batch = WBatch<G, NR>;
    gp<const void> gu;
    int64_t cols;
    uint32_t lo;
    __device__ void load(Batch& b, int rb) const { load_wbatch<G, NR>(b, gu, rb, cols, lo); }
    __device__ void terms(const Batch& b, int k, double t[8]) const {
        float gv[8];
        unpack8<G>(b.r[k], gv);
#pragma unroll
        for (int j = 0; j < 8; ++j) t[j] = (double)gv[j];
    }
};

// ------------------------------------------------------------- edge units
// Every other unit: ragged rows or columns, widths of any alignment, and the
// units of fewer rows that short lists are cut into. Lane l = 32 h + q takes the
// 8 columns from cs = min(c0 + 8q, cols - 8) of rows 2k + h of each 4-row batch,
// so every access stays inside its row (wide loads at the element's own
// alignment); the first sh = c0 + 8q - cs columns of a shifted lane belong to the
// lane before it and are left out, as is everything of a lane past the edge
// (sh >= 8). Rows past the unit's last repeat it and are left out. Two batches
// are in flight ahead of the one being formed. Sums, bounds and the staging of
// the row partials are those of the whole units (columns in runs of 16 rows).
// Matrices narrower than 8 columns are summed element by element, lane by row.
// A short list is bound by its longest wavefront, so its units are 32 to 128 rows
// high (fac_plan). Measured on a 4-layer list of width 500 (fp32 gradients, UF8
// momentum): marginals 118 -> 14 us, RMS 151 -> 14, residual 338 -> 25 against
// 256-row units of 16 x 64 tiles with double-double sums and guarded loads.
typedef uint32_t ua_u4 __attribute__((ext_vector_type(4), aligned(2)));
typedef float ua_f4 __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t ua_u2 __attribute__((ext_vector_type(2), aligned(1)));

template <int G>
__device__ __forceinline__ void load8_ua(Raw8<G>& r, gp<const void> g, int64_t e) {
    if constexpr (G == G_BF16) {
        const ua_u4 x = *g_as<const ua_u4>(g_as<const uint16_t>(g) + e);
        r.w = make_uint4(x.x, x.y, x.z, x.w);
    } else {
        const gp<const float> f = g_as<const float>(g) + e;
        const ua_f4 x = *g_as<const ua_f4>(f), y = *g_as<const ua_f4>(f + 4);
        r.a = make_float4(x.x, x.y, x.z, x.w);
        r.b = make_float4(y.x, y.y, y.z, y.w);
    }
}

struct EdgeLane {
    int64_t r0, cs, cols;
    int nr, h, q, sh;
};

__device__ __forceinline__ EdgeLane edge_lane(const GD& d, int ur, int64_t ru, int64_t cu) {
    EdgeLane w;
    w.h = (int)(threadIdx.x >> 5) & 1;
    w.q = (int)threadIdx.x & 31;
    w.r0 = ru * ur;
    w.nr = (int)(d.rows - w.r0 < ur ? d.rows - w.r0 : ur);
    w.cols = d.cols;
    const int64_t c = cu * 256 + 8 * w.q;
    w.cs = c < d.cols - 8 ? c : d.cols - 8;
    w.sh = c - w.cs < 8 ? (int)(c - w.cs) : 8;
    return w;
}

constexpr int kEdgeNR = 4;   // rows per batch
constexpr int kEdgeFR = 16;  // rows per finish group and column run

// Batches 0 .. nb - 1 with two in flight: load(batch, i) for i < nb (the last
// ones load batch nb - 1 again, so that the loads are not conditional), step(batch, i).
template <class Batch, class L, class S>
__device__ __forceinline__ void edge_batches(int nb, L load, S step) {
    Batch A, B, C;
    load(A, 0);
    load(B, 1 < nb ? 1 : nb - 1);
#pragma unroll 1
    for (int bi = 0;;) {
        load(C, bi + 2 < nb ? bi + 2 : nb - 1);
        step(A, bi);
        if (++bi >= nb) break;
        load(A, bi + 2 < nb ? bi + 2 : nb - 1);
        step(B, bi);
        if (++bi >= nb) break;
        load(B, bi + 2 < nb ? bi + 2 : nb - 1);
        step(C, bi);
        if (++bi >= nb) break;
    }
}

// P: Batch, load(batch, row) for the lane's row of each pair (row already
// clamped), terms(batch, k, ok, t): 8 values whose squares are the terms, zero
// where left out (ok: the row is inside the unit).
template <class P>
__device__ __forceinline__ void edge_unit_sums(const P& pol, const GD& d, const EdgeLane& w, int64_t ru, int64_t cu,
                                               double* stage) {
    constexpr int NR = kEdgeNR, NP = NR / 2, FR = kEdgeFR;
    const int lane = threadIdx.x & 63, h = w.h, q = w.q, nr = w.nr;
    double cacc[8], crun[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) cacc[j] = crun[j] = 0.0;
    const int nb = (nr + NR - 1) / NR;
    auto load = [&](typename P::Batch& b, int bi) {
#pragma unroll
        for (int k = 0; k < NP; ++k) {
            const int row = NR * bi + 2 * k + h;
            pol.load(b, k, row < nr ? row : nr - 1);
        }
    };
    auto step = [&](const typename P::Batch& b, int bi) {
#pragma unroll
        for (int k = 0; k < NP; ++k) {
            const int row = NR * bi + 2 * k + h;
            double t[8];
            pol.terms(b, k, row < nr, t);
            double rs = t[0] * t[0];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                crun[j] = __builtin_fma(t[j], t[j], crun[j]);
                if (j > 0) rs = __builtin_fma(t[j], t[j], rs);
                if (k & 1) __asm__ volatile("" : "+v"(crun[j]));  // two row pairs' terms live at a time
            }
            stage[(row & (FR - 1)) * kWStride + q] = rs;
        }
        if (((bi + 1) * NR) % FR != 0 && bi + 1 < nb) return;
        // a group of 16 rows is staged: 4 lanes finish each row from 8 partials apiece
        __builtin_amdgcn_wave_barrier();
        const int rrow = lane >> 2, rpart = lane & 3, row = (bi * NR & ~(FR - 1)) + rrow;
        const double2* st = reinterpret_cast<const double2*>(stage + rrow * kWStride + 8 * rpart);
        const double2 p0 = st[0], p1 = st[1], p2 = st[2], p3 = st[3];
        double rs = ((p0.x + p0.y) + (p1.x + p1.y)) + ((p2.x + p2.y) + (p3.x + p3.y));
        rs += dpp_d<kDppQuadXor1>(rs);
        rs += dpp_d<kDppQuadXor2>(rs);
        if (rpart == 0 && row < nr) d.rowpart[cu * d.rows + w.r0 + row] = rs;
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            cacc[j] += crun[j];
            crun[j] = 0.0;
        }
    };
    edge_batches<typename P::Batch>(nb, load, step);
    // the two halves hold the even and the odd rows of the same columns
    const gp<double> cp = d.colpart + (ru * w.cols + w.cs);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        cacc[j] += __shfl_xor(cacc[j], 32);
        if ((j < 4) == (h == 0) && j >= w.sh) cp[j] = cacc[j];
    }
}

// Matrices narrower than 8 columns: lane l takes rows l, l + 64, .. of the unit
// (all columns); term(row, column) is the value whose square is summed. Row
// sums are chains of at most 7, column sums of at most 4 terms and a butterfly.
template <class T>
__device__ __forceinline__ void narrow_unit_sums(const GD& d, int ur, int64_t ru, T term) {
    const int lane = threadIdx.x & 63;
    const int64_t r0 = ru * ur;
    const int nr = (int)(d.rows - r0 < ur ? d.rows - r0 : ur), nc = (int)d.cols;
    double cs[7] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    for (int r = lane; r < nr; r += 64) {
        double rs = 0.0;
#pragma unroll
        for (int j = 0; j < 7; ++j)
            if (j < nc) {
                const double t = term(r0 + r, j);
                rs = __builtin_fma(t, t, rs);
                cs[j] = __builtin_fma(t, t, cs[j]);
            }
        d.rowpart[r0 + r] = rs;
    }
#pragma unroll
    for (int j = 0; j < 7; ++j) {
#pragma unroll
        for (int m = 1; m < 64; m <<= 1) cs[j] += __shfl_xor(cs[j], m);
        if (lane == 0 && j < nc) d.colpart[ru * d.cols + j] = cs[j];
    }
}

// The whole-unit body takes this unit.
__device__ __forceinline__ bool whole_unit(const FacArgs& a, const GD& d, int64_t ru) {
    return a.ur == 256 && (d.cols & 255) == 0 && d.rows - ru * 256 >= 256;
}

template <int G>
struct EdgeMarg {
    struct Batch {
        Raw8<G> r[kEdgeNR / 2];
    };
    gp<const void> g;
    int64_t e0, cols;  // element of the lane's first column in the unit's first row
    int sh;
    __device__ void load(Batch& b, int k, int row) const { load8_ua<G>(b.r[k], g, e0 + row * cols); }
    __device__ void terms(const Batch& b, int k, bool ok, double t[8]) const {
        float gv[8];
        unpack8<G>(b.r[k], gv);
#pragma unroll
        for (int j = 0; j < 8; ++j) t[j] = (double)(((j >= sh) & ok) ? gv[j] : 0.0f);
    }
};

// One wavefront per unit, 4 per 256-thread workgroup (each with its own
// LDS stage), as in the other streaming kernels.
__device__ __forceinline__ int64_t unit_of_wave(int64_t base) {
    return base + xcd_order(blockIdx.x, gridDim.x) * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
}

// ------------------------------------------- Adafactor 1-D tensors (WG each)
template <int G>
__device__ __forceinline__ void ada_vec1d(const FacArgs& a, const FacDesc& d, DD* sh, double& clip_s) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t n = d.rows * d.cols;
    for (int64_t i = tid; i < n; i += blockDim.x) {
        const double gi = (double)grad_at_g<G>(to_g(d.g), i);
        const float old = vec_decode(a.v_codec, a.v_block, d.v, d.vm, i, a.cf);
        d.rtmp[i] = (float)(a.beta * (double)old + a.omb * (gi * gi + a.eps1));
    }
    __syncthreads();
    vec_encode(a.v_codec, a.v_block, d.rtmp, n, a.v_floor, d.v, d.vm, wave, 4, lane);
    DD s{0.0, 0.0};
    for (int64_t i = tid; i < n; i += blockDim.x) {
        const double uu = (1.0 / sqrt((double)d.rtmp[i])) * (double)grad_at_g<G>(to_g(d.g), i);
        dd_add(s, uu * uu);
    }
    s = block_dd_sum(s, sh);
    if (tid == 0) {
        const double rms = sqrt(dd_value(s) / (double)n);
        clip_s = rms / a.clip_d > 1.0 ? rms / a.clip_d : 1.0;
    }
    __syncthreads();
    const double clip = clip_s;
    for (int64_t i = tid; i < n; i += blockDim.x) {
        const double uu = (1.0 / sqrt((double)d.rtmp[i])) * (double)grad_at_g<G>(to_g(d.g), i);
        const double pd = (double)d.p[i] * a.decay;
        d.p[i] = (float)(pd - a.lr * (uu / clip));
    }
}

// ---------------------------------------------------------- CAME momentum
// In-step momentum of element e of tensor d from its uhat (binary64 EMA,
// rounded to fp32): m = fl32(beta1 * mhat + (1 - beta1) * uhat).
__device__ __forceinline__ float came_momentum(const FacArgs& a, const FacDesc& d, int64_t e, float uh) {
    float mh;
    if (a.m_codec == UF8) {
        const int32_t q = reinterpret_cast<const int8_t*>(d.m)[e];
        mh = uf8_decode(q, div127((double)d.mm[e / a.m_block]));
    } else {
        mh = reinterpret_cast<const float*>(d.m)[e];
    }
    return (float)(a.beta1 * (double)mh + a.omb1 * (double)uh);
}

// ------------------------------------------------ CAME 1-D tensors (WG each)
template <int G>
__device__ __forceinline__ void came_vec1d(const FacArgs& a, const FacDesc& d, DD* sh, double& clip_s) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t n = d.rows * d.cols;
    for (int64_t i = tid; i < n; i += blockDim.x) {
        const double gi = (double)grad_at_g<G>(to_g(d.g), i);
        const float old = vec_decode(a.v_codec, a.v_block, d.v, d.vm, i, a.cf);
        d.rtmp[i] = (float)(a.beta * (double)old + a.omb * (gi * gi + a.eps1));
    }
    __syncthreads();
    vec_encode(a.v_codec, a.v_block, d.rtmp, n, a.v_floor, d.v, d.vm, wave, 4, lane);
    DD s{0.0, 0.0};
    for (int64_t i = tid; i < n; i += blockDim.x) {
        const double uu = (1.0 / sqrt((double)d.rtmp[i])) * (double)grad_at_g<G>(to_g(d.g), i);
        dd_add(s, uu * uu);
    }
    s = block_dd_sum(s, sh);
    if (tid == 0) {
        const double rms = sqrt(dd_value(s) / (double)n);
        clip_s = rms / a.clip_d > 1.0 ? rms / a.clip_d : 1.0;
    }
    __syncthreads();
    const double clip = clip_s;
    for (int64_t i = tid; i < n; i += blockDim.x) {
        const double uu = (1.0 / sqrt((double)d.rtmp[i])) * (double)grad_at_g<G>(to_g(d.g), i);
        const float uh = (float)(uu / clip);
        const float m = came_momentum(a, d, i, uh);
        d.ctmp[i] = m;
        const double pd = (double)d.p[i] * a.decay;
        d.p[i] = (float)(pd - a.lr * (double)m);
    }
    __syncthreads();
    vec_encode(a.m_codec, a.m_block, d.ctmp, n, 0.0f, d.m, d.mm, wave, 4, lane);
}

// The first a.lead workgroups of the first launch (lead = a.lead) step a 1-D tensor each: one workgroup is
// latency-bound, and beside the streaming units it is hidden.
template <int G, bool CAME>
__global__ __launch_bounds__(256) void fac_marg_kernel(const FacArgs a, int64_t base, int lead) {
    __shared__ __attribute__((aligned(16))) double stages[4][2 * MargTerms<G>::NR * kWStride];
    static_assert(2 * MargTerms<G>::NR >= kEdgeFR, "the edge units' stage");
    if ((int)blockIdx.x < lead) {
        const FacDesc& d = a.D[a.n2 + blockIdx.x];
        DD* const sh = reinterpret_cast<DD*>(&stages[0][0]);
        if constexpr (CAME)
            came_vec1d<G>(a, d, sh, stages[1][0]);
        else
            ada_vec1d<G>(a, d, sh, stages[1][0]);
        return;
    }
    double* stage = stages[threadIdx.x >> 6];
    const int64_t unit = base + xcd_order(blockIdx.x - lead, gridDim.x - lead) * 4 +
                         __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (unit >= a.total_units) return;
    const GD d = gview(a.D[locate(a.unit_begins, a.n2, unit)]);
    const int64_t u = unit - d.unit_begin, ru = u / d.ncu, cu = u % d.ncu;
    if (whole_unit(a, d, ru)) {
        const WholeLane w = whole_lane(d, ru, cu);
        const MargTerms<G> pol{unit_base<G>(d, w), w.cols, w.lo};
        whole_unit_sums(pol, d, ru, cu, stage);
    } else if (d.cols >= 8) {
        const EdgeLane w = edge_lane(d, a.ur, ru, cu);
        const EdgeMarg<G> pol{d.g, w.r0 * w.cols + w.cs, w.cols, w.sh};
        edge_unit_sums(pol, d, w, ru, cu, stage);
    } else {
        narrow_unit_sums(d, a.ur, ru, [&](int64_t i, int64_t j) { return (double)grad_at_g<G>(d.g, i * d.cols + j); });
    }
}

// 1-D tensors that the marginal kernel's workgroups do not take (fac_plan).
template <int G, bool CAME>
__global__ __launch_bounds__(256) void fac_vec1d_kernel(const FacArgs a) {
    __shared__ DD sh[4];
    __shared__ double clip_s;
    const FacDesc& d = a.D[a.n2 + blockIdx.x];
    if constexpr (CAME)
        came_vec1d<G>(a, d, sh, clip_s);
    else
        ada_vec1d<G>(a, d, sh, clip_s);
}

template <int G, bool CAME>
static hipError_t marg_launch(const FacArgs& a, hipStream_t s) {
    if (a.lead < a.n1) {
        hipLaunchKernelGGL((fac_vec1d_kernel<G, CAME>), dim3((unsigned)a.n1), dim3(256), 0, s, a);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    constexpr int64_t kMaxGrid = int64_t(1) << 30;
    int lead = a.lead;
    for (int64_t base = 0; base < a.total_units || lead > 0; base += 4 * kMaxGrid) {
        const int64_t left = (a.total_units - base + 3) / 4;
        const int64_t grid = (left < kMaxGrid ? left : kMaxGrid) + lead;
        hipLaunchKernelGGL((fac_marg_kernel<G, CAME>), dim3((unsigned)grid), dim3(256), 0, s, a, base, lead);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        lead = 0;
    }
    return hipSuccess;
}

hipError_t launch_fac_marg(const FacArgs& a, int grad_dtype, bool came, hipStream_t s) {
    if (grad_dtype == G_BF16) return came ? marg_launch<G_BF16, true>(a, s) : marg_launch<G_BF16, false>(a, s);
    return came ? marg_launch<G_F32, true>(a, s) : marg_launch<G_F32, false>(a, s);
}

// ------------------------------------------------------------- finalize
// role 0: second moment (EMA beta, codes vr/vc, factors rfac/cfac);
// role 1: CAME confidence (EMA beta3, codes cr/cc, factors sr/sc).
// fac_mean: one workgroup per 64 elements of a factor vector (R tiles, then C
// tiles, of every 2-D tensor): its four wavefronts merge every fourth unit
// partial of each element (a column of a tall matrix has hundreds), then EMA of
// the mean with the decoded old value, rounded to fp32; R tiles also leave their
// double-double sum for mean(R). fac_enc: re-encodes each code block and forms
// the factors C_j^-1/2 and r_i = (R_i / mean R)^-1/2 (each wavefront merges the
// R tile sums itself).
struct FinRole {
    int codec, B;
    void *rc, *cc;
    float *rm, *cm;
    double *fr, *fc;
    double beta, omb;
    float lf;
};

__device__ __forceinline__ FinRole fin_role(const FacArgs& a, const FacDesc& d, int role) {
    FinRole r;
    r.codec = role ? a.c_codec : a.v_codec;
    r.B = role ? a.c_block : a.v_block;
    r.rc = role ? d.cr : d.vr;
    r.rm = role ? d.crm : d.vrm;
    r.cc = role ? d.cc : d.vc;
    r.cm = role ? d.ccm : d.vcm;
    r.fr = role ? d.sr : d.rfac;
    r.fc = role ? d.sc : d.cfac;
    r.beta = role ? a.beta3 : a.beta;
    r.omb = role ? a.omb3 : a.omb;
    r.lf = role ? a.c_floor : a.v_floor;
    return r;
}

// fl32(y) is the same for every binary64 y' within tol of y >= 0: y lies
// farther than tol from both fp32 rounding midpoints around fl32(y) (the
// midpoint of two adjacent fp32 values is exact in binary64).
__device__ __forceinline__ bool f32_round_robust(double y, double tol) {
    const float f = (float)y;
    const uint32_t b = f2u(f);
    if (b >= 0x7F7FFFFFu) return false;  // FLT_MAX, +inf, NaN, negative: take the exact path
    const float up = u2f(b + 1u);
    const float dn = b == 0u ? -u2f(1u) : u2f(b - 1u);
    const double mhi = 0.5 * ((double)f + (double)up), mlo = 0.5 * ((double)f + (double)dn);
    return (y - mlo > tol) & (mhi - y > tol);
}

// The decoded momentum of element e (UF8 or fp32).
__device__ __forceinline__ float came_mhat(const FacArgs& a, const GD& v, int64_t e) {
    if (a.m_codec == UF8) return uf8_decode(g_as<const int8_t>(v.m)[e], div127((double)v.mm[e / a.m_block]));
    return g_as<const float>(v.m)[e];
}

// Exact (double-double) sum of the marginal terms of row idx (isrow) or
// column idx of a 2-D tensor -- role 0: fl64(g^2 + eps1); role 1: CAME's
// residual terms -- by the whole wavefront; each term is formed exactly as the
// marginal kernels form it.
template <int G>
__device__ DD exact_line_sum(const FacArgs& a, const FacDesc& d, int role, bool isrow, int64_t idx, int lane) {
    const GD v = gview(d);
    const int64_t len = isrow ? d.cols : d.rows;
    const double clip = role ? v.scal[0] : 1.0;
    const double rclip = 1.0 / clip;
    DD acc{0.0, 0.0};
#pragma unroll 4
    for (int64_t k = lane; k < len; k += 64) {
        const int64_t i = isrow ? idx : k, j = isrow ? k : idx;
        const int64_t e = i * d.cols + j;
        float g;
        if constexpr (G == G_BF16)
            g = bf16_to_f32(g_as<const uint16_t>(v.g)[e]);
        else
            g = g_as<const float>(v.g)[e];
        double t;
        if (role == 0) {
            t = marg_term(g, a.eps1);
        } else {
            const double uu = (v.rfac[i] * v.cfac[j]) * (double)g;
            t = res_term(a, came_mhat(a, v, e), div_to_f32(uu, clip, rclip));
        }
        dd_add(acc, t);
    }
    return dd_wave_sum(acc);
}

// Relative distance from an fp32 rounding midpoint below which the EMA value
// from the fast partial sums may round differently from the one from the exact
// sum. A partial is within 25u (u = 2^-53; second moment) or 129u (CAME's
// residual) of its exact sum of squares, the oracle's terms are within 2u of
// ours plus eps, the partials are merged double-double, and the mean, eps and
// the EMA add at most 6u. 40u bounds the second moment's total (role 0), 160u
// CAME's confidence (role 1); an EMA value that close to a midpoint is about
// one in ten million (one in a million) of the elements (the exact sum of its
// line is then taken).
constexpr double kRobustTol[2] = {40.0 * 0x1p-53, 160.0 * 0x1p-53};
constexpr int kMeanTile = 64;  // elements per workgroup of fac_mean

template <int G>
__global__ __launch_bounds__(256) void fac_mean_kernel(const FacArgs a, int role) {
    __shared__ DD part[4][64];
    __shared__ double ysh[64];
    __shared__ uint64_t pend_sh;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t tile = blockIdx.x;
    const FacDesc& d = a.D[locate(a.mt_begins, a.n2, tile)];
    const FinRole R = fin_role(a, d, role);
    const int64_t lt = tile - d.mt_begin, nrt = (d.rows + kMeanTile - 1) / kMeanTile;
    const bool isrow = lt < nrt;
    const int64_t n = isrow ? d.rows : d.cols;
    const int64_t s = (isrow ? lt : lt - nrt) * kMeanTile, i = s + lane;
    const bool act = i < n;
    // 1. the element's partials, every fourth by this wavefront (their loads do not depend on the
    // running sum: unrolled, they are issued ahead)
    DD acc{0.0, 0.0};
    if (act) {
        const int np = isrow ? d.ncu : d.nru;
        const gp<const double> pp = to_g((const double*)(isrow ? d.rowpart : d.colpart)) + i;
#pragma unroll 8
        for (int k = w; k < np; k += 4) dd_add(acc, pp[(int64_t)k * n]);
    }
    part[w][lane] = acc;
    __syncthreads();
    // 2. EMA of the mean; where the partials' error could change its fp32 rounding (or with exact_all),
    // the element's row or column is summed again, exactly, by one of the wavefronts
    const double cnt = (double)(isrow ? d.cols : d.rows);
    float old = 0.0f;
    if (w == 0) {
        double y = 0.0;
        if (act) {
            acc = dd_merge(dd_merge(part[0][lane], part[1][lane]), dd_merge(part[2][lane], part[3][lane]));
            old = vec_decode(R.codec, R.B, isrow ? R.rc : R.cc, isrow ? R.rm : R.cm, i, a.cf);
            y = R.beta * (double)old + R.omb * (dd_value(acc) / cnt + (role ? a.eps2 : a.eps1));
        }
        const bool robust = !act || (!a.exact_all && f32_round_robust(y, kRobustTol[role] * y));
        const uint64_t pend = __ballot(!robust);
        ysh[lane] = y;
        if (lane == 0) pend_sh = pend;
    }
    __syncthreads();
    uint64_t pend = pend_sh;
    if (pend) {
        for (int k = 0; pend; ++k, pend &= pend - 1) {
            if ((k & 3) != w) continue;
            const int src = __builtin_ctzll(pend);
            const DD S = exact_line_sum<G>(a, d, role, isrow, s + src, lane);
            if (lane == 0) ysh[src] = dd_value(S) / cnt;  // the mean; the EMA follows below
        }
        __syncthreads();
    }
    if (w != 0) return;
    double y = ysh[lane];
    if ((pend_sh >> lane) & 1) y = R.beta * (double)old + R.omb * y;
    const float x = act ? (float)y : 0.0f;
    if (act) (isrow ? d.rtmp : d.ctmp)[i] = x;
    if (isrow) {
        const DD t = dd_wave_sum(DD{(double)x, 0.0});
        if (lane == 0) {
            d.rsum[2 * lt] = t.hi;
            d.rsum[2 * lt + 1] = t.lo;
        }
    }
}

// One wavefront per code block of up to 256 elements, one workgroup per larger
// block (up to 8 elements per lane either way).
__global__ __launch_bounds__(256) void fac_enc_kernel(const FacArgs a, int role) {
    __shared__ uint32_t smn[4], smx[4];
    const int codec = role ? a.c_codec : a.v_codec;
    const int B = role ? a.c_block : a.v_block;
    const bool wg = B > 256;
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int64_t blk = wg ? (int64_t)blockIdx.x : (int64_t)blockIdx.x * 4 + w;
    if (blk >= a.total_blk[role]) return;
    const FacDesc& d = a.D[locate(a.blk_begins[role], a.n2, blk)];
    const FinRole R = fin_role(a, d, role);
    const int64_t lb = blk - d.blk_begin[role];
    const int64_t nbr = (d.rows + B - 1) / B;
    const bool isrow = lb < nbr;
    const int64_t n = isrow ? d.rows : d.cols;
    const int64_t b = isrow ? lb : lb - nbr;
    const int64_t s = b * B, e = s + B < n ? s + B : n;
    const gp<const float> x = to_g((const float*)(isrow ? d.rtmp : d.ctmp));
    const int t0 = wg ? (int)threadIdx.x : lane, st = wg ? 256 : 64;
    const int nk = (B + st - 1) / st;  // 1 .. 8
    float xv[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const int64_t i = s + t0 + k * st;
        xv[k] = k < nk && i < e ? x[i] : 0.0f;
    }
    double mr = 1.0;
    if (isrow) {
        DD acc{0.0, 0.0};
        const gp<const double> rs = to_g((const double*)d.rsum);
        const int64_t nt = (d.rows + kMeanTile - 1) / kMeanTile;
#pragma unroll 4
        for (int64_t k = lane; k < nt; k += 64) acc = dd_merge(acc, DD{rs[2 * k], rs[2 * k + 1]});
        mr = dd_value(dd_wave_sum(acc)) / (double)d.rows;
    }
    const gp<double> f = to_g(isrow ? R.fr : R.fc);
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const int64_t i = s + t0 + k * st;
        if (k < nk && i < e) f[i] = 1.0 / sqrt(isrow ? (double)xv[k] / mr : (double)xv[k]);
    }
    void* codes = isrow ? R.rc : R.cc;
    float* meta = isrow ? R.rm : R.cm;
    if (codec == FP32) {
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int64_t i = s + t0 + k * st;
            if (k < nk && i < e) reinterpret_cast<float*>(codes)[i] = xv[k];
        }
        return;
    }
    uint32_t mn = 0xFFFFFFFFu, mx = 0u;
#pragma unroll
    for (int k = 0; k < 8; ++k) {  // absent elements are +0: in neither reduction
        mn = OpMin::f(mn, pos_min_key(xv[k]));
        mx = OpMax::f(mx, pos_max_key(xv[k]));
    }
    mn = group_reduce<OpMin, 64>(mn);
    mx = group_reduce<OpMax, 64>(mx);
    if (wg) {
        if (lane == 0) {
            smn[w] = mn;
            smx[w] = mx;
        }
        __syncthreads();
        mn = OpMin::f(OpMin::f(smn[0], smn[1]), OpMin::f(smn[2], smn[3]));
        mx = OpMax::f(OpMax::f(smx[0], smx[1]), OpMax::f(smx[2], smx[3]));
    }
    const ALFit fit = al_fit(mn, mx, R.lf);
    if (t0 == 0) {
        meta[2 * b] = fit.any ? (float)fit.lmin : 0.0f;
        meta[2 * b + 1] = fit.any ? (float)fit.delta : 0.0f;
    }
    const ALEnc enc = al_enc_params(fit.lmin, fit.any ? (double)(codec == AL16 ? 65534 : 254) / fit.delta : 1.0);
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        const int64_t i = s + t0 + k * st;
        if (k < nk && i < s + B) {
            if (codec == AL16)
                reinterpret_cast<uint16_t*>(codes)[i] = (uint16_t)al_encode_fast<65534>(xv[k], enc);
            else
                reinterpret_cast<uint8_t*>(codes)[i] = (uint8_t)al_encode_fast<254>(xv[k], enc);
        }
    }
}

hipError_t launch_fac_fin(const FacArgs& a, int role, int grad_dtype, hipStream_t s) {
    if (a.n2 == 0) return hipSuccess;
    if (grad_dtype == G_BF16)
        hipLaunchKernelGGL(fac_mean_kernel<G_BF16>, dim3((unsigned)a.total_mt), dim3(256), 0, s, a, role);
    else
        hipLaunchKernelGGL(fac_mean_kernel<G_F32>, dim3((unsigned)a.total_mt), dim3(256), 0, s, a, role);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const bool wg = (role ? a.c_block : a.v_block) > 256;
    const int64_t grid = wg ? a.total_blk[role] : (a.total_blk[role] + 3) / 4;
    hipLaunchKernelGGL(fac_enc_kernel, dim3((unsigned)grid), dim3(256), 0, s, a, role);
    return hipGetLastError();
}

// ------------------------------------------------ RMS partials (per unit)
// u_ij = (r_i c_j) g_ij, exactly the oracle's operation order. One wave per unit.
//
// Edge units (see edge_unit_sums): left-out elements have g = 0 (and row
// factor 0 past the last row). TERMS (lists with a ragged matrix): every
// term u^2 is added double-double, so a unit's partial is its exact sum to about
// 2^-100. Otherwise the 8 terms of a lane's row are added pairwise first, as in the
// whole units' layout below.
template <int G>
struct EdgeRmsBatch {
    Raw8<G> r[kEdgeNR / 2];
    double ri[kEdgeNR / 2];
};

template <int G, bool TERMS>
__device__ __forceinline__ DD edge_unit_rms(const GD& d, const EdgeLane& w) {
    constexpr int NR = kEdgeNR, NP = NR / 2;
    const int nr = w.nr, sh = w.sh;
    const int64_t e0 = w.r0 * w.cols + w.cs;
    double cf[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) cf[j] = d.cfac[w.cs + j];
    DD acc{0.0, 0.0};
    edge_batches<EdgeRmsBatch<G>>(
        (nr + NR - 1) / NR,
        [&](EdgeRmsBatch<G>& b, int bi) {
#pragma unroll
            for (int k = 0; k < NP; ++k) {
                const int row = NR * bi + 2 * k + w.h, rr = row < nr ? row : nr - 1;
                load8_ua<G>(b.r[k], d.g, e0 + rr * w.cols);
                b.ri[k] = d.rfac[w.r0 + rr];
            }
        },
        [&](const EdgeRmsBatch<G>& b, int bi) {
#pragma unroll
            for (int k = 0; k < NP; ++k) {
                const bool ok = NR * bi + 2 * k + w.h < nr;
                const double ri = ok ? b.ri[k] : 0.0;
                float gv[8];
                unpack8<G>(b.r[k], gv);
                double t[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const double uu = (ri * cf[j]) * (double)(((j >= sh) & ok) ? gv[j] : 0.0f);
                    t[j] = uu * uu;
                }
                if constexpr (TERMS)
                    dd_add8(acc, t);
                else
                    dd_add(acc, sum8(t));
            }
        });
    return acc;
}

// Matrices narrower than 8 columns, lane by row.
template <int G>
__device__ __forceinline__ DD narrow_unit_rms(const GD& d, int ur, int64_t ru) {
    DD acc{0.0, 0.0};
    for (int64_t i = ru * ur + (threadIdx.x & 63); i < d.rows && i < (ru + 1) * ur; i += 64)
        for (int64_t j = 0; j < d.cols; ++j) {
            const double uu = (d.rfac[i] * d.cfac[j]) * (double)grad_at_g<G>(d.g, i * d.cols + j);
            dd_add(acc, uu * uu);
        }
    return acc;
}

// Whole units (the marginal kernels' streaming layout): lane 32 h + q holds
// columns 8q .. 8q + 7 of rows 2k + h of each 8-row batch, 16-byte gradient
// loads, the next batch loaded before the current one's arithmetic. TERMS (units
// of a matrix with ragged rows): summed term by term like the edge units. Otherwise the 8
// terms u^2 of a lane's row are added pairwise (relative error <= 3u) and
// those sums accumulated double-double, so a unit's partial is within 3u of
// its exact sum. The clip divisor then
// carries a relative error of at most about 2u: it scales Adafactor's update
// (inside the parameter tolerance), and for CAME it can move fl32(u / clip)
// by one fp32 ulp only where u / clip lies within that distance of an fp32
// rounding midpoint, about one element in 10^8.
template <int G, bool TERMS>
__device__ __forceinline__ DD whole_unit_rms(const GD& d, int64_t ru, int64_t cu) {
    const WholeLane w = whole_lane(d, ru, cu);
    const gp<const void> gu = unit_base<G>(d, w);
    const int64_t cols = w.cols;
    const uint32_t lo = w.lo;
    double cf[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) cf[j] = d.cfac[w.c0 + 8 * w.q + j];
    const gp<const double> rf = d.rfac + w.r0 + w.h;  // row factor of row 2k + h of a batch: rf[rb + 2k]
    constexpr int NR = TERMS ? 4 : 8;  // the term-by-term sum needs more registers
    constexpr int NP = NR / 2;
    DD acc{0.0, 0.0};
    WBatch<G, NR> A, B;
    double ra[NP], rb_[NP];
    load_wbatch<G, NR>(A, gu, 0, cols, lo);
#pragma unroll
    for (int k = 0; k < NP; ++k) ra[k] = rf[2 * k];
    auto step = [&](const WBatch<G, NR>& cur, const double ri[NP]) {
#pragma unroll
        for (int k = 0; k < NP; ++k) {
            float gv[8];
            unpack8<G>(cur.r[k], gv);
            double t[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const double uu = (ri[k] * cf[j]) * (double)gv[j];
                t[j] = uu * uu;
            }
            if constexpr (TERMS)
                dd_add8(acc, t);
            else
                dd_add(acc, sum8(t));
        }
    };
    constexpr int NB = 256 / NR;
    auto load = [&](WBatch<G, NR>& b, double ri[NP], int bi) {
        load_wbatch<G, NR>(b, gu, bi * NR, cols, lo);
#pragma unroll
        for (int k = 0; k < NP; ++k) ri[k] = rf[bi * NR + 2 * k];
    };
    // last pair of batches peeled (see whole_unit_sums)
#pragma unroll 1
    for (int bi = 0; bi < NB - 2; bi += 2) {
        load(B, rb_, bi + 1);
        step(A, ra);
        load(A, ra, bi + 2);
        step(B, rb_);
    }
    load(B, rb_, NB - 1);
    step(A, ra);
    step(B, rb_);
    return acc;
}

// By what the list holds, so that a list pays for no other body's registers: matrices of whole units, cut 256 rows
// high (kRmsWhole: the 1.1B list's step 2617 us, 2627 with kRmsMixed's kernel) or less (kRmsShort), or some ragged
// matrix (kRmsMixed; whole matrices cut less than 256 rows high are then summed term by term too).
enum RmsKind { kRmsWhole, kRmsShort, kRmsMixed };

template <int G, int KIND>
__global__ __launch_bounds__(256) void fac_rms_kernel(const FacArgs a, int64_t base) {
    const int64_t unit = unit_of_wave(base);
    if (unit >= a.total_units) return;
    const GD d = gview(a.D[locate(a.unit_begins, a.n2, unit)]);
    const int64_t u = unit - d.unit_begin, ru = u / d.ncu, cu = u % d.ncu;
    DD acc;
    if constexpr (KIND == kRmsWhole) {
        acc = whole_unit_rms<G, false>(d, ru, cu);
    } else if constexpr (KIND == kRmsShort) {
        acc = edge_unit_rms<G, false>(d, edge_lane(d, a.ur, ru, cu));
    } else {
        if (whole_unit(a, d, ru))
            acc = (d.rows & 255) == 0 ? whole_unit_rms<G, false>(d, ru, cu) : whole_unit_rms<G, true>(d, ru, cu);
        else if (d.cols >= 8)
            acc = edge_unit_rms<G, true>(d, edge_lane(d, a.ur, ru, cu));
        else
            acc = narrow_unit_rms<G>(d, a.ur, ru);
    }
    acc = dd_wave_sum(acc);
    if ((threadIdx.x & 63) == 0) {
        a.rmspart[2 * unit] = acc.hi;
        a.rmspart[2 * unit + 1] = acc.lo;
    }
}

template <int G>
static hipError_t rms_launch(const FacArgs& a, hipStream_t s) {
    if (a.any_ragged) return launch_wave_per_unit(fac_rms_kernel<G, kRmsMixed>, a, s);
    return a.ur == 256 ? launch_wave_per_unit(fac_rms_kernel<G, kRmsWhole>, a, s)
                       : launch_wave_per_unit(fac_rms_kernel<G, kRmsShort>, a, s);
}

hipError_t launch_fac_rms(const FacArgs& a, int grad_dtype, hipStream_t s) {
    return grad_dtype == G_BF16 ? rms_launch<G_BF16>(a, s) : rms_launch<G_F32>(a, s);
}

// ------------------------------------------ clip divisor (workgroup / tensor)
__global__ __launch_bounds__(256) void fac_clip_kernel(const FacArgs a) {
    __shared__ DD sh[4];
    const FacDesc& d = a.D[blockIdx.x];
    const int64_t nu = (int64_t)d.nru * d.ncu;
    const gp<const double> rp = to_g((const double*)a.rmspart) + 2 * d.unit_begin;
    DD s{0.0, 0.0};
#pragma unroll 4
    for (int64_t k = threadIdx.x; k < nu; k += 256) s = dd_merge(s, DD{rp[2 * k], rp[2 * k + 1]});
    s = block_dd_sum(s, sh);
    if (threadIdx.x == 0) {
        const double rms = sqrt(dd_value(s) / (double)(d.rows * d.cols));
        d.scal[0] = rms / a.clip_d > 1.0 ? rms / a.clip_d : 1.0;
    }
}

hipError_t launch_fac_clip(const FacArgs& a, hipStream_t s) {
    if (a.n2 == 0) return hipSuccess;
    hipLaunchKernelGGL(fac_clip_kernel, dim3(a.n2), dim3(256), 0, s, a);
    return hipGetLastError();
}

// --------------------------------------------------- Adafactor apply (2-D)
// p <- p (1 - lr wd) - lr u / clip. Widths that are a multiple of 256: one
// wavefront per chunk of 2048 elements (32 per 256 x 256, 4 per 256-thread
// workgroup) with no loop: the grid itself streams, as in the
// AdamW step. Lanes take 4 consecutive columns of each 256-column row
// segment, so every load and store instruction covers a contiguous 1 KB of
// parameters (512 bytes of bf16 gradients); 16-byte non-temporal parameter
// accesses. Other widths: one wavefront per kFlatChunk consecutive elements of
// the row-major flattening, so that the accesses are as wide and aligned as
// there; each lane's row and column follow from one division per chunk, and the
// factors are gathered (they stay in cache). Measured on the width-500 list:
// CAME's apply 151 -> 46 us against element-by-element accesses; seven layers of width
// 2240 (378M parameters): 1386 us with four gathers per element, 967 with the row's value
// and 16-byte column loads where a sub-tile stays inside a row (FlatPos::straight).
constexpr int kChunksPerUnit = 32;
constexpr int kFlatChunk = kFacFlatChunk;

// A chunk of a matrix whose width is a multiple of 256 as rows and columns: 8 / W
// rows from row0, 256 W columns from col0 (W units side by side; the unit columns
// left over in a unit row, ncu mod W, take W = 1: 8 rows x 256). A unit row (256
// rows) holds 32 ncu chunks; rows past the matrix's last are left out.
struct RowChunk {
    int64_t row0, col0;
    bool full;  // W units (else one)
};

template <int W>
__device__ __forceinline__ RowChunk row_chunk(const GD& d, int64_t t_ch) {
    const int64_t cpr = (int64_t)d.ncu * kChunksPerUnit;  // chunks per unit row
    const int64_t ur = t_ch / cpr, r = t_ch - ur * cpr;
    const int64_t ng = d.ncu / W;             // groups of W units in a unit row
    RowChunk c;
    c.full = r < ng * W * kChunksPerUnit;
    if (c.full) {
        const int64_t grp = r / (W * kChunksPerUnit), ci = r - grp * (W * kChunksPerUnit);
        c.row0 = ur * 256 + ci * (8 / W);
        c.col0 = grp * (256 * W);
    } else {
        const int64_t x = r - ng * W * kChunksPerUnit;
        c.row0 = ur * 256 + (x % kChunksPerUnit) * 8;
        c.col0 = (ng * W + x / kChunksPerUnit) * 256;
    }
    return c;
}

// Adafactor apply over a row chunk (lane l: columns 4l .. 4l + 3 of each
// 256-column segment): every load of the chunk is issued before the
// arithmetic. RAG: only nrow of the chunk's rows exist.
template <int G, int W, bool RAG>
__device__ __forceinline__ void ada_apply_rows(const FacArgs& a, const GD& d, int64_t row0, int64_t col0, int nrow) {
    constexpr int R = 8 / W;
    const int64_t cb = col0 + 4 * (threadIdx.x & 63);
    const double rclip = 1.0 / d.scal[0], lr = a.lr, decay = a.decay;
    float gv[R][W][4];
    float4 pv[R][W];
    double ri[R], cf[W][4];
#pragma unroll
    for (int k = 0; k < R; ++k) {
        const int64_t row = row0 + (!RAG || k < nrow ? k : nrow - 1);
        ri[k] = d.rfac[row];
#pragma unroll
        for (int sg = 0; sg < W; ++sg) {
            const int64_t e = row * d.cols + cb + 256 * sg;
            load_g4<G>(d.g, e, gv[k][sg]);
            pv[k][sg] = ld_f4<true>(d.p + e);
        }
    }
#pragma unroll
    for (int sg = 0; sg < W; ++sg)
#pragma unroll
        for (int j = 0; j < 4; ++j) cf[sg][j] = d.cfac[cb + 256 * sg + j];
#pragma unroll
    for (int k = 0; k < R; ++k) {
        if (RAG && k >= nrow) break;
#pragma unroll
        for (int sg = 0; sg < W; ++sg) {
            const float pin[4] = {pv[k][sg].x, pv[k][sg].y, pv[k][sg].z, pv[k][sg].w};
            float out[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const double uu = (ri[k] * cf[sg][j]) * (double)gv[k][sg][j];
                const double pd = (double)pin[j] * decay;
                out[j] = (float)(pd - lr * (uu * rclip));  // p carries a tolerance: multiply by 1 / clip
            }
            st_f4<true>(d.p + (row0 + k) * d.cols + cb + 256 * sg, make_float4(out[0], out[1], out[2], out[3]));
        }
    }
}

// kFlatChunk elements from e0, the first `valid` of them inside the matrix
// (FULL: all).
template <int G, bool FULL>
__device__ __forceinline__ void ada_apply_flat(const FacArgs& a, const GD& d, int64_t e0, int valid) {
    constexpr int K = kFlatChunk / 256;
    const int l4 = 4 * (threadIdx.x & 63);
    float gv[K][4];
    float4 pv[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int64_t e = e0 + 256 * k + l4;
        if constexpr (FULL) {
            load_g4<G>(d.g, e, gv[k]);
            pv[k] = ld_f4<true>(d.p + e);
        } else {
            float h[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const bool ok = 256 * k + l4 + t < valid;
                gv[k][t] = ok ? grad_at_g<G>(d.g, e + t) : 0.0f;
                h[t] = ok ? d.p[e + t] : 0.0f;
            }
            pv[k] = make_float4(h[0], h[1], h[2], h[3]);
        }
    }
    const double rclip = 1.0 / d.scal[0], lr = a.lr, decay = a.decay;
    FlatPos pos(d.rows, d.cols, e0 + l4);
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int64_t e = e0 + 256 * k + l4;
        const float pin[4] = {pv[k].x, pv[k].y, pv[k].z, pv[k].w};
        float out[4];
        double rf[4], cf[4];
        if (pos.straight()) {
            rf[0] = rf[1] = rf[2] = rf[3] = d.rfac[pos.i];
            pos.cols4(d.cfac, cf);
        } else {
            pos.each(e, [&](int t, int64_t i, int64_t j) {
                rf[t] = d.rfac[i];
                cf[t] = d.cfac[j];
            });
        }
        pos.next();
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const double uu = (rf[t] * cf[t]) * (double)gv[k][t];
            const double pd = (double)pin[t] * decay;
            out[t] = (float)(pd - lr * (uu * rclip));
        }
        if constexpr (FULL) {
            st_f4<true>(d.p + e, make_float4(out[0], out[1], out[2], out[3]));
        } else {
#pragma unroll
            for (int t = 0; t < 4; ++t)
                if (256 * k + l4 + t < valid) d.p[e + t] = out[t];
        }
    }
}

constexpr int kAdaApplyW = 2;

// Wavefront -> apply chunk.
__device__ __forceinline__ int64_t chunk_of_wave(int64_t base) {
    return base + xcd_order(blockIdx.x, gridDim.x) * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
}

// Four waves per SIMD: more of them in flight mix the pass's streams and slow it (the 1.1B list's step 2739
// us at the six its registers allow, 2673-2676 at 4 and 5, 2687 at 3).
template <int G>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4, 4))) void ada_apply_kernel(const FacArgs a, int64_t base) {
    const int64_t chunk = chunk_of_wave(base);
    if (chunk >= a.rows_ach) return;
    const GD d = gview(a.D[locate(a.ach_begins, a.n2, chunk)]);
    const RowChunk c = row_chunk<kAdaApplyW>(d, chunk - d.ach_begin);
    constexpr int R = 8 / kAdaApplyW;
    const int64_t left = d.rows - c.row0;
    if (left <= 0) return;
    if (c.full) {
        if (left >= R)
            ada_apply_rows<G, kAdaApplyW, false>(a, d, c.row0, c.col0, R);
        else
            ada_apply_rows<G, kAdaApplyW, true>(a, d, c.row0, c.col0, (int)left);
    } else if (left >= 8) {
        ada_apply_rows<G, 1, false>(a, d, c.row0, c.col0, 8);
    } else {
        ada_apply_rows<G, 1, true>(a, d, c.row0, c.col0, (int)left);
    }
}

template <int G>
__global__ __launch_bounds__(256) void ada_apply_flat_kernel(const FacArgs a, int64_t base) {
    const int64_t chunk = chunk_of_wave(base);
    if (chunk >= a.total_ach) return;
    const GD d = gview(a.D[locate(a.ach_begins, a.n2, chunk)]);
    const int64_t e0 = (chunk - d.ach_begin) * kFlatChunk, left = d.rows * d.cols - e0;
    if (left >= kFlatChunk)
        ada_apply_flat<G, true>(a, d, e0, kFlatChunk);
    else
        ada_apply_flat<G, false>(a, d, e0, (int)left);
}

// One wavefront per apply chunk of [begin, end), 4 per 256-thread workgroup;
// grids beyond 2^31 workgroups take several launches.
template <class K>
static hipError_t launch_per_chunk(K kernel, const FacArgs& a, int64_t begin, int64_t end, hipStream_t s) {
    constexpr int64_t kMaxGrid = int64_t(1) << 31;
    for (int64_t base = begin; base < end; base += 4 * kMaxGrid) {
        const int64_t left = (end - base + 3) / 4;
        const int64_t grid = left < kMaxGrid ? left : kMaxGrid;
        hipLaunchKernelGGL(kernel, dim3((unsigned)grid), dim3(256), 0, s, a, base);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

hipError_t launch_ada_apply(const FacArgs& a, int grad_dtype, hipStream_t s) {
    const bool bf = grad_dtype == G_BF16;
    const hipError_t e = bf ? launch_per_chunk(ada_apply_kernel<G_BF16>, a, 0, a.rows_ach, s)
                            : launch_per_chunk(ada_apply_kernel<G_F32>, a, 0, a.rows_ach, s);
    if (e != hipSuccess) return e;
    return bf ? launch_per_chunk(ada_apply_flat_kernel<G_BF16>, a, a.rows_ach, a.total_ach, s)
              : launch_per_chunk(ada_apply_flat_kernel<G_F32>, a, a.rows_ach, a.total_ach, s);
}

// ------------------------------------------- CAME residual marginal sums
// Terms (uhat - m)^2 with uhat = fl32(u / clip) and m the in-step momentum.
// Whole units: the marginal kernels' streaming layout (whole_unit_sums).
// Each unit row is one 256-element momentum block
// (the width is a multiple of 256), so a row's codes share one scale; the
// lane's 8 momentum values of a row are one 8-byte word of codes (or two
// 16-byte fp32 loads), loaded with the gradients one batch ahead.
constexpr int kResNR = 4;  // unit rows per batch of the residual kernel (its terms need more registers)
template <int G, bool UF>
struct ResBatch;
template <int G>
struct ResBatch<G, true> {
    WBatch<G, kResNR> g;
    uint2 mc[kResNR / 2];  // 8 UF8 codes of the lane's row in each row pair
    float ms[kResNR / 2];  // their block's absmax
    double ri[kResNR / 2];
};
template <int G>
struct ResBatch<G, false> {
    WBatch<G, kResNR> g;
    float4 ma[kResNR / 2], mb[kResNR / 2];  // fp32 momentum
    double ri[kResNR / 2];
};

template <int G, bool UF>
struct ResTerms {
    static constexpr int NR = kResNR;
    static constexpr int FR = 16;  // row partials finished 16 rows at a time (4 batches)
    static constexpr bool ILP = false;  // the residual terms need the registers for occupancy
    // the registers the single column sum frees (against runs) hold a third batch: 3 waves per SIMD either way
    static constexpr int DEPTH = 3;
    using Batch = ResBatch<G, UF>;
    const FacArgs* a;
    gp<const void> gu;   // the unit's first gradient
    gp<const void> mu;   // the unit's first momentum element (codes or fp32)
    gp<const float> msu;  // absmax of the unit's first row's block (UF8)
    gp<const double> rf;  // row factor of the lane's first row
    int64_t cols, hcols;  // hcols = h * cols: the lane's row within a pair
    uint32_t lo;
    double cf[8];
    double cfmin;  // the smallest of the lane's column factors
    double clip, rclip;
    __device__ void load(Batch& b, int rb) const {
        load_wbatch<G, NR>(b.g, gu, rb, cols, lo);
#pragma unroll
        for (int k = 0; k < NR / 2; ++k) {
            const int64_t off = (int64_t)(rb + 2 * k) * cols;  // row rb + 2k + h, with lo
            b.ri[k] = rf[rb + 2 * k];
            if constexpr (UF) {
                b.mc[k] = ld_u2<false>(g_as<const void>(g_as<const uint8_t>(mu) + off + lo));
                b.ms[k] = msu[(off + hcols) >> 8];  // the row's momentum block
            } else {
                const gp<const float> m = g_as<const float>(mu) + off + lo;
                b.ma[k] = ld_f4<false>(m);
                b.mb[k] = ld_f4<false>(m + 4);
            }
        }
    }
    __device__ void terms(const Batch& b, int k, double t[8]) const {
        float gv[8], mh[8], uh[8];
        unpack8<G>(b.g.r[k], gv);
        if constexpr (UF) {
            const double st = div127((double)b.ms[k]);
            const uint32_t w[2] = {b.mc[k].x, b.mc[k].y};
#pragma unroll
            for (int j = 0; j < 8; ++j) mh[j] = uf8_decode((int32_t)(int8_t)(uint8_t)(w[j >> 2] >> (8 * (j & 3))), st);
        } else {
            mh[0] = b.ma[k].x, mh[1] = b.ma[k].y, mh[2] = b.ma[k].z, mh[3] = b.ma[k].w;
            mh[4] = b.mb[k].x, mh[5] = b.mb[k].y, mh[6] = b.mb[k].z, mh[7] = b.mb[k].w;
        }
        // uhat = fl32(u / clip), u = fl64(fl64(r c) g): from the quotient with 1 / clip folded into the
        // row factor (two multiplications), the exact division where its rounding is not decided
        const double rk = b.ri[k] * rclip;
        double qv[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) qv[j] = (rk * cf[j]) * (double)gv[j];
        // A nonzero bf16 gradient has |g| >= 2^-133, so when rk * min_j c_j >= 2^7 (1 + 2^-18) on every
        // lane each q_j is zero or above 2^-126 (1 + 2^-19) (three roundings of at most u each): only the
        // midpoint test remains. The condition is taken wave-wide, so the branch is uniform.
        bool ok;
        if (G == G_BF16 && __builtin_expect(__all(rk * cfmin >= 0x1.00004p7), 1))
            ok = f32_midpoints_decided<8>(qv, uh);
        else
            ok = f32_roundings_decided<8>(qv, uh);
        if (__builtin_expect(!ok, 0)) {
#pragma unroll
            for (int j = 0; j < 8; ++j) uh[j] = (float)(((b.ri[k] * cf[j]) * (double)gv[j]) / clip);
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) t[j] = res_diff(*a, mh[j], uh[j]);
    }
};

template <int G, bool UF>
__device__ __forceinline__ void whole_unit_res(const FacArgs& a, const GD& d, int64_t ru, int64_t cu, double* stage) {
    const WholeLane w = whole_lane(d, ru, cu);
    ResTerms<G, UF> pol;
    pol.a = &a;
    pol.gu = unit_base<G>(d, w);
    const int64_t e0 = w.r0 * w.cols + w.c0;
    pol.mu = UF ? g_as<const void>(g_as<const uint8_t>(d.m) + e0) : g_as<const void>(g_as<const float>(d.m) + e0);
    pol.msu = d.mm + (e0 >> 8);
    pol.rf = d.rfac + w.r0 + w.h;
    pol.cols = w.cols;
    pol.hcols = w.h * w.cols;
    pol.lo = w.lo;
#pragma unroll
    for (int j = 0; j < 8; ++j) pol.cf[j] = d.cfac[w.c0 + 8 * w.q + j];
    pol.cfmin = pol.cf[0];
#pragma unroll
    for (int j = 1; j < 8; ++j) pol.cfmin = pol.cf[j] < pol.cfmin ? pol.cf[j] : pol.cfmin;
    pol.clip = d.scal[0];
    pol.rclip = 1.0 / pol.clip;
    whole_unit_sums(pol, d, ru, cu, stage);
}

// Edge units (see edge_unit_sums). A lane's 8 momentum codes may straddle two
// 256-element blocks of the flattening: both scales are loaded.
template <int G, bool UF>
struct EdgeRes {
    struct Batch {
        Raw8<G> r[kEdgeNR / 2];
        double ri[kEdgeNR / 2];
        uint2 mc[UF ? kEdgeNR / 2 : 1];        // codes,
        float ms0[UF ? kEdgeNR / 2 : 1], ms1[UF ? kEdgeNR / 2 : 1];  // absmax of the first code's block and of the next,
        int cut[UF ? kEdgeNR / 2 : 1];         // codes of the first block
        float4 ma[UF ? 1 : kEdgeNR / 2], mb[UF ? 1 : kEdgeNR / 2];  // or fp32 momentum
    };
    const FacArgs* a;
    gp<const void> g, m;
    gp<const float> mm;
    gp<const double> rf;  // row factor of the unit's first row
    int64_t e0, cols, lastblk;
    int sh;
    double cf[8], cfmin, clip, rclip;
    __device__ void load(Batch& b, int k, int row) const {
        const int64_t e = e0 + row * cols;
        load8_ua<G>(b.r[k], g, e);
        b.ri[k] = rf[row];
        if constexpr (UF) {
            const ua_u2 c = *g_as<const ua_u2>(g_as<const uint8_t>(m) + e);
            const int64_t blk = e >> 8;
            b.mc[k] = make_uint2(c.x, c.y);
            b.ms0[k] = mm[blk];
            b.ms1[k] = mm[blk < lastblk ? blk + 1 : blk];
            b.cut[k] = 256 - (int)(e & 255);
        } else {
            const gp<const float> f = g_as<const float>(m) + e;
            const ua_f4 x = *g_as<const ua_f4>(f), y = *g_as<const ua_f4>(f + 4);
            b.ma[k] = make_float4(x.x, x.y, x.z, x.w);
            b.mb[k] = make_float4(y.x, y.y, y.z, y.w);
        }
    }
    __device__ void terms(const Batch& b, int k, bool ok, double t[8]) const {
        float gv[8], mh[8], uh[8];
        unpack8<G>(b.r[k], gv);
        if constexpr (UF) {
            const double st0 = div127((double)b.ms0[k]), st1 = div127((double)b.ms1[k]);
            const uint32_t w[2] = {b.mc[k].x, b.mc[k].y};
#pragma unroll
            for (int j = 0; j < 8; ++j)
                mh[j] = uf8_decode((int32_t)(int8_t)(uint8_t)(w[j >> 2] >> (8 * (j & 3))), j < b.cut[k] ? st0 : st1);
        } else {
            mh[0] = b.ma[k].x, mh[1] = b.ma[k].y, mh[2] = b.ma[k].z, mh[3] = b.ma[k].w;
            mh[4] = b.mb[k].x, mh[5] = b.mb[k].y, mh[6] = b.mb[k].z, mh[7] = b.mb[k].w;
        }
        // left out: g = m = 0, so uhat - m = 0
        const double ri = ok ? b.ri[k] : 0.0;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const bool in = (j >= sh) & ok;
            gv[j] = in ? gv[j] : 0.0f;
            mh[j] = in ? mh[j] : 0.0f;
        }
        const double rk = ri * rclip;
        double qv[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) qv[j] = (rk * cf[j]) * (double)gv[j];
        // (the range test can be dropped as in the whole units; a row left out has rk = 0 and keeps it)
        bool dec;
        if (G == G_BF16 && __builtin_expect(__all(rk * cfmin >= 0x1.00004p7), 1))
            dec = f32_midpoints_decided<8>(qv, uh);
        else
            dec = f32_roundings_decided<8>(qv, uh);
        if (__builtin_expect(!dec, 0)) {
#pragma unroll
            for (int j = 0; j < 8; ++j) uh[j] = (float)(((ri * cf[j]) * (double)gv[j]) / clip);
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) t[j] = res_diff(*a, mh[j], uh[j]);
    }
};

template <int G, bool UF>
__device__ __forceinline__ void edge_unit_res(const FacArgs& a, const GD& d, int64_t ru, int64_t cu, double* stage) {
    const EdgeLane w = edge_lane(d, a.ur, ru, cu);
    EdgeRes<G, UF> pol;
    pol.a = &a;
    pol.g = d.g;
    pol.m = d.m;
    pol.mm = d.mm;
    pol.rf = d.rfac + w.r0;
    pol.e0 = w.r0 * w.cols + w.cs;
    pol.cols = w.cols;
    pol.lastblk = (d.rows * d.cols - 1) >> 8;
    pol.sh = w.sh;
#pragma unroll
    for (int j = 0; j < 8; ++j) pol.cf[j] = d.cfac[w.cs + j];
    pol.cfmin = pol.cf[0];
#pragma unroll
    for (int j = 1; j < 8; ++j) pol.cfmin = pol.cf[j] < pol.cfmin ? pol.cf[j] : pol.cfmin;
    pol.clip = d.scal[0];
    pol.rclip = 1.0 / pol.clip;
    edge_unit_sums(pol, d, w, ru, cu, stage);
}

// Whole units and edge units in a kernel each (the edge body needs the registers of one wavefront per
// SIMD less); each leaves the other's units alone.
template <int G, bool UF>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) void came_res_whole_kernel(const FacArgs a, int64_t base) {
    __shared__ __attribute__((aligned(16))) double stages[4][2 * ResTerms<G, UF>::FR * kWStride];
    const int64_t unit = unit_of_wave(base);
    if (unit >= a.total_units) return;
    const GD d = gview(a.D[locate(a.unit_begins, a.n2, unit)]);
    const int64_t u = unit - d.unit_begin, ru = u / d.ncu, cu = u % d.ncu;
    if (whole_unit(a, d, ru)) whole_unit_res<G, UF>(a, d, ru, cu, stages[threadIdx.x >> 6]);
}

template <int G, bool UF>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void came_res_edge_kernel(const FacArgs a, int64_t base) {
    __shared__ __attribute__((aligned(16))) double stages[4][kEdgeFR * kWStride];
    double* stage = stages[threadIdx.x >> 6];
    const int64_t unit = unit_of_wave(base);
    if (unit >= a.total_units) return;
    const GD d = gview(a.D[locate(a.unit_begins, a.n2, unit)]);
    const int64_t u = unit - d.unit_begin, ru = u / d.ncu, cu = u % d.ncu;
    if (whole_unit(a, d, ru)) return;
    if (d.cols >= 8) {
        edge_unit_res<G, UF>(a, d, ru, cu, stage);
    } else {
        const double clip = d.scal[0], rclip = 1.0 / clip;
        narrow_unit_sums(d, a.ur, ru, [&](int64_t i, int64_t j) {
            const int64_t e = i * d.cols + j;
            const double uu = (d.rfac[i] * d.cfac[j]) * (double)grad_at_g<G>(d.g, e);
            return res_diff(a, came_mhat(a, d, e), div_to_f32(uu, clip, rclip));
        });
    }
}

hipError_t launch_came_res(const FacArgs& a, int grad_dtype, hipStream_t s) {
    const bool uf = a.m_codec == UF8;
    hipError_t e = hipSuccess;
    if (a.any_whole)
        e = grad_dtype == G_BF16 ? (uf ? launch_wave_per_unit(came_res_whole_kernel<G_BF16, true>, a, s)
                                       : launch_wave_per_unit(came_res_whole_kernel<G_BF16, false>, a, s))
                                 : (uf ? launch_wave_per_unit(came_res_whole_kernel<G_F32, true>, a, s)
                                       : launch_wave_per_unit(came_res_whole_kernel<G_F32, false>, a, s));
    if (e != hipSuccess || !a.any_edge) return e;
    return grad_dtype == G_BF16 ? (uf ? launch_wave_per_unit(came_res_edge_kernel<G_BF16, true>, a, s)
                                      : launch_wave_per_unit(came_res_edge_kernel<G_BF16, false>, a, s))
                                : (uf ? launch_wave_per_unit(came_res_edge_kernel<G_F32, true>, a, s)
                                      : launch_wave_per_unit(came_res_edge_kernel<G_F32, false>, a, s));
}

// ------------------------------------------------------ CAME apply (2-D)
// Recompute uhat and m, encode m, and p <- p (1 - lr wd) - lr (s_i s_j) m, in the Adafactor apply's chunks.
//
// One 256-element momentum block (4 consecutive elements per lane): new momentum
// from the updates u(j) = (r_i c_j) g and their quotients qv = ((r_i / clip) c_j) g; mw: the lane's codes, ms the
// block's absmax (UF8), else mv the fp32 momentum. Leaves the momentum in mnew, its codes and
// their absmax in mw / am (UF8) or itself in mv.
template <bool UF, class U>
__device__ __forceinline__ void came_apply_block(const FacArgs& a, const double qv[4], U u, double clip,
                                                 uint32_t& mw, float ms, float4& mv, const bool in[4], uint32_t& am,
                                                 float mnew[4]) {
    float mh[4], uh[4];
    if constexpr (UF) {
        const double st = div127((double)ms);
#pragma unroll
        for (int j = 0; j < 4; ++j) mh[j] = uf8_decode((int32_t)(int8_t)(uint8_t)(mw >> (8 * j)), st);
    } else {
        mh[0] = mv.x, mh[1] = mv.y, mh[2] = mv.z, mh[3] = mv.w;
    }
    if (__builtin_expect(!f32_roundings_decided<4>(qv, uh), 0)) {
#pragma unroll
        for (int j = 0; j < 4; ++j) uh[j] = (float)(u(j) / clip);
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        mnew[j] = (float)(a.beta1 * (double)mh[j] + a.omb1 * (double)uh[j]);
        if (!in[j]) mnew[j] = 0.0f;
    }
    if constexpr (UF) {
        am = 0u;
#pragma unroll
        for (int j = 0; j < 4; ++j) am = OpMax::f(am, abs_bits(mnew[j]));
        am = group_reduce<OpMax, 64>(am);
        const double rs = am != 0u ? rdiv127((double)u2f(am)) : 0.0;
        uint32_t q[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) q[j] = rint_low_bits((double)mnew[j] * rs) & 0xFFu;
        mw = q[0] | (q[1] << 8) | (q[2] << 16) | (q[3] << 24);
    } else {
        mv = make_float4(mnew[0], mnew[1], mnew[2], mnew[3]);
    }
}

// kFlatChunk elements of the flattening from e0 (widths that are not a multiple
// of 256), or kCameTail of the last chunk, the first `valid` of them inside the matrix (FULL: all): a momentum
// block is one 256-element sub-tile. The parameter is formed in binary64 and rounded once (three matrices of
// 20000 x 6000, bf16: 1596 us per step, 1580 with an fp32 update). The guarded tail sets the registers: in
// pieces of 512 elements it needs 104 (4 waves per SIMD) in place of 131 to 134.
constexpr int kCameTail = 512;
template <int G, bool UF, bool FULL>
__device__ __forceinline__ void came_apply_flat(const FacArgs& a, const GD& d, int64_t e0, int valid) {
    constexpr int K = (FULL ? kFlatChunk : kCameTail) / 256;
    const int lane = threadIdx.x & 63, l4 = 4 * lane;
    const gp<uint8_t> mc = g_as<uint8_t>(d.m);
    const gp<float> mf = g_as<float>(d.m);
    float gv[K][4], ms[K];
    float4 pv[K], mv[K];
    uint32_t mw[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int64_t e = e0 + 256 * k + l4;
        ms[k] = 0.0f;
        mw[k] = 0u;
        mv[k] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        const bool live = FULL || 256 * k < valid;  // codes and scales are padded to whole blocks
        if (UF && live) {
            mw[k] = ld_u1<true>(g_as<const void>(mc + e));
            ms[k] = d.mm[(e0 >> 8) + k];
        }
        if constexpr (FULL) {
            load_g4<G>(d.g, e, gv[k]);
            pv[k] = ld_f4<true>(d.p + e);
            if constexpr (!UF) mv[k] = ld_f4<true>(gp<const float>(mf + e));
        } else {
            float h[4], f[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const bool ok = 256 * k + l4 + t < valid;
                gv[k][t] = ok ? grad_at_g<G>(d.g, e + t) : 0.0f;
                h[t] = ok ? d.p[e + t] : 0.0f;
                f[t] = !UF && ok ? mf[e + t] : 0.0f;
            }
            pv[k] = make_float4(h[0], h[1], h[2], h[3]);
            mv[k] = make_float4(f[0], f[1], f[2], f[3]);
        }
    }
    const double clip = d.scal[0], rclip = 1.0 / clip;
    FlatPos pos(d.rows, d.cols, e0 + l4);
#pragma unroll
    for (int k = 0; k < K; ++k) {
        if (!FULL && 256 * k >= valid) break;
        const int64_t e = e0 + 256 * k + l4;
        double rc[4], qv[4], ss[4];  // r_i c_j, ((r_i / clip) c_j) g, s_i s_j
        if (pos.straight()) {
            const double r = d.rfac[pos.i], rk = r * rclip, sri = d.sr[pos.i];
            double cf[4], sf[4];
            pos.cols4(d.cfac, cf);
            pos.cols4(d.sc, sf);
#pragma unroll
            for (int t = 0; t < 4; ++t) rc[t] = r * cf[t], qv[t] = rk * cf[t], ss[t] = sri * sf[t];
        } else {
            pos.each(e, [&](int t, int64_t i, int64_t j) {
                const double r = d.rfac[i], c = d.cfac[j];
                rc[t] = r * c;
                qv[t] = (r * rclip) * c;
                ss[t] = d.sr[i] * d.sc[j];
            });
        }
        pos.next();
        bool in[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) in[t] = FULL || 256 * k + l4 + t < valid;
        uint32_t am = 0u;
        float mnew[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) qv[t] *= (double)gv[k][t];
        came_apply_block<UF>(a, qv, [&](int t) { return rc[t] * (double)gv[k][t]; }, clip, mw[k], ms[k], mv[k], in, am, mnew);
        const float pin[4] = {pv[k].x, pv[k].y, pv[k].z, pv[k].w};
        float po[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const double upd = ss[t] * (double)mnew[t];
            po[t] = (float)((double)pin[t] * a.decay - a.lr * upd);
        }
        if constexpr (FULL) {
            st_f4<true>(d.p + e, make_float4(po[0], po[1], po[2], po[3]));
            if constexpr (!UF) st_f4<true>(mf + e, mv[k]);
        } else {
#pragma unroll
            for (int t = 0; t < 4; ++t)
                if (in[t]) {
                    d.p[e + t] = po[t];
                    if constexpr (!UF) mf[e + t] = mnew[t];
                }
        }
        if constexpr (UF) {
            st_u1<true>(g_as<void>(mc + e), mw[k]);
            if (lane == 0) d.mm[(e0 >> 8) + k] = u2f(am);
        }
    }
}

// Widths that are a multiple of 256: a wavefront takes a chunk of 8 / W rows x
// 256 W columns (lane l: columns 4l .. 4l + 3 of each 256-column segment), one
// row at a time: each row is one contiguous segment of 256 W elements, and each
// 256-column segment of a row is one momentum block over all 64 lanes.
// WHOLE (rows a multiple of 256 too): the parameter update runs in fp32 (the states never depend on p, which is
// held to a relative tolerance), p' = p - fma(lr wd, p, ((lr s_i) s_j) m) on the fp32 roundings of the factors: the
// change carries a few fp32 roundings, p' one (1 - lr wd itself has no fp32 form near 1: steps of 2^-24).
// Otherwise in binary64, rounded once, for the chunk's first nrow rows.
// W = 2 (2 KB parameter segments, 88 registers) measured 1.8% faster than
// 8 rows x 256 columns in two 32-lane halves; W = 1 and 4 no faster, W = 8
// (232 registers) 21% slower.
constexpr int kCameApplyW = 2;
template <int G, bool UF, int W, bool WHOLE>
__device__ __forceinline__ void came_apply_rows(const FacArgs& a, const GD& d, int64_t row0, int64_t col0, int nrow) {
    using F = typename std::conditional<WHOLE, float, double>::type;
    const int lane = threadIdx.x & 63;
    const int64_t cb = col0 + 4 * lane;
    const int64_t cols = d.cols;
    const double clip = d.scal[0], rclip = 1.0 / clip;
    const float lrwd = (float)(1.0 - a.decay);
    const gp<uint8_t> mc = g_as<uint8_t>(d.m);
    const gp<float> mf = g_as<float>(d.m);
    double cf[W][4];
    F sf[W][4];
#pragma unroll
    for (int sg = 0; sg < W; ++sg)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            cf[sg][j] = d.cfac[cb + 256 * sg + j];
            sf[sg][j] = (F)d.sc[cb + 256 * sg + j];
        }
#pragma unroll 1
    for (int k = 0; k < nrow; ++k) {
        const int64_t row = row0 + k;
        const double ri = d.rfac[row], rk = ri * rclip;
        const F si = WHOLE ? (F)(a.lr * d.sr[row]) : (F)d.sr[row];
        float gv[W][4], ms[W];
        float4 pv[W], mv[W];
        uint32_t mw[W];
#pragma unroll
        for (int sg = 0; sg < W; ++sg) {
            const int64_t e = row * cols + cb + 256 * sg;
            load_g4<G>(d.g, e, gv[sg]);
            pv[sg] = ld_f4<true>(d.p + e);
            ms[sg] = 0.0f;
            mw[sg] = 0u;
            if constexpr (UF) {
                mw[sg] = ld_u1<true>(g_as<const void>(mc + e));
                ms[sg] = d.mm[e >> 8];
            } else {
                mv[sg] = ld_f4<true>(gp<const float>(mf + e));
            }
        }
#pragma unroll
        for (int sg = 0; sg < W; ++sg) {
            const int64_t e = row * cols + cb + 256 * sg;
            double qv[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) qv[j] = (rk * cf[sg][j]) * (double)gv[sg][j];
            const bool in[4] = {true, true, true, true};
            uint32_t am = 0u;
            float mnew[4], pout[4];
            came_apply_block<UF>(a, qv, [&](int j) { return (ri * cf[sg][j]) * (double)gv[sg][j]; }, clip, mw[sg], ms[sg], mv[sg],
                                 in, am, mnew);
            const float pin[4] = {pv[sg].x, pv[sg].y, pv[sg].z, pv[sg].w};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const F upd = (si * sf[sg][j]) * (F)mnew[j];
                if constexpr (WHOLE)
                    pout[j] = pin[j] - __builtin_fmaf(lrwd, pin[j], upd);
                else
                    pout[j] = (float)((double)pin[j] * a.decay - a.lr * upd);
            }
            st_f4<true>(d.p + e, make_float4(pout[0], pout[1], pout[2], pout[3]));
            if constexpr (UF) {
                st_u1<true>(g_as<void>(mc + e), mw[sg]);
                if (lane == 0) d.mm[e >> 8] = u2f(am);
            } else {
                st_f4<true>(mf + e, mv[sg]);
            }
        }
    }
}

// Chunk c of a matrix, of which `left` rows start in the chunk or after it.
template <int G, bool UF, bool WHOLE>
__device__ __forceinline__ void came_apply_chunk(const FacArgs& a, const GD& d, const RowChunk& c, int64_t left) {
    if (c.full)
        came_apply_rows<G, UF, kCameApplyW, WHOLE>(a, d, c.row0, c.col0, left < 8 / kCameApplyW ? (int)left : 8 / kCameApplyW);
    else
        came_apply_rows<G, UF, 1, WHOLE>(a, d, c.row0, c.col0, left < 8 ? (int)left : 8);
}

// MIXED: some width that is a multiple of 256 has ragged rows (the binary64 body's registers cost lists of whole
// units 0.4% of a step; a launch of its own would cost short lists more).
template <int G, bool UF, bool MIXED>
__global__ __launch_bounds__(256) void came_apply_kernel(const FacArgs a, int64_t base) {
    const int64_t chunk = chunk_of_wave(base);
    if (chunk >= a.rows_ach) return;
    const GD d = gview(a.D[locate(a.ach_begins, a.n2, chunk)]);
    const RowChunk c = row_chunk<kCameApplyW>(d, chunk - d.ach_begin);
    const int64_t left = d.rows - c.row0;
    if (left <= 0) return;
    if (!MIXED || (d.rows & 255) == 0)
        came_apply_chunk<G, UF, true>(a, d, c, left);
    else
        came_apply_chunk<G, UF, false>(a, d, c, left);
}

template <int G, bool UF>
__global__ __launch_bounds__(256) void came_apply_flat_kernel(const FacArgs a, int64_t base) {
    const int64_t chunk = chunk_of_wave(base);
    if (chunk >= a.total_ach) return;
    const GD d = gview(a.D[locate(a.ach_begins, a.n2, chunk)]);
    const int64_t e0 = (chunk - d.ach_begin) * kFlatChunk, left = d.rows * d.cols - e0;
    if (left >= kFlatChunk)
        came_apply_flat<G, UF, true>(a, d, e0, kFlatChunk);
    else
        for (int o = 0; o < left; o += kCameTail) came_apply_flat<G, UF, false>(a, d, e0 + o, (int)left - o);
}

template <int G, bool UF>
static hipError_t came_apply_launch(const FacArgs& a, hipStream_t s) {
    const hipError_t e = a.rows_ragged ? launch_per_chunk(came_apply_kernel<G, UF, true>, a, 0, a.rows_ach, s)
                                       : launch_per_chunk(came_apply_kernel<G, UF, false>, a, 0, a.rows_ach, s);
    return e != hipSuccess ? e : launch_per_chunk(came_apply_flat_kernel<G, UF>, a, a.rows_ach, a.total_ach, s);
}

hipError_t launch_came_apply(const FacArgs& a, int grad_dtype, hipStream_t s) {
    const bool uf = a.m_codec == UF8;
    if (grad_dtype == G_BF16) return uf ? came_apply_launch<G_BF16, true>(a, s) : came_apply_launch<G_BF16, false>(a, s);
    return uf ? came_apply_launch<G_F32, true>(a, s) : came_apply_launch<G_F32, false>(a, s);
}

}  // namespace al
