// Standalone block codecs (gfx950): AL8 / AL16 quantize and dequantize
// (section 4.1, Eq. al_bounds, al_quant, al_dequant; section 4.2) and the
// uniform signed 8-bit code UF8 (section 4.3).
//
// A wavefront owns a chunk of max(B, 256 K) consecutive elements, 4 per lane in
// each 256-element sub-tile, all of its loads issued before the arithmetic and
// each byte touched once. K = 8 where that fills the chip: the per-block scalar
// work of a chunk (binary64 divisions and endpoint logarithms) then runs once, one
// block per lane pair, for up to 32 blocks at a time; short arrays take K = 1 for
// more wavefronts.
#include "al_device.hpp"
#include "al_internal.hpp"

namespace al {

// The decode polynomial's coefficients, read with scalar loads.
__constant__ Exp2Coef kExp2Codec = AL_EXP2_TAYLOR;

const Exp2Coef& exp2_coef() {
    static const Exp2Coef c = AL_EXP2_TAYLOR;
    return c;
}


// Encode parameters of blocks smaller than a sub-tile, in LDS.
struct BlockEnc {
    ALEnc e;
};

// One chunk of K sub-tiles from element e0, the first `valid` elements inside the
// array (FULL: all).
template <int C, int B, int K, bool NT, bool FULL>
__device__ __forceinline__ void quantize_chunk(gp<const float> x, int64_t e0, int valid, int lane, float log_floor,
                                               gp<uint8_t> codes, gp<float> meta, uint2* skey, BlockEnc* senc) {
    constexpr int NB = 256 * K / B;               // blocks
    constexpr int GL = B < kSub ? B / 4 : 64;     // lanes per block within a sub-tile
    constexpr int PER = B < kSub ? kSub / B : 1;  // blocks per sub-tile
    constexpr int SUBS = B < kSub ? 1 : B / kSub; // sub-tiles per block
    float xv[K][4];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int rel = k * kSub + 4 * lane;
        if constexpr (FULL) {
            const float4 t = ld_f4<NT>(x + e0 + rel);
            xv[k][0] = t.x, xv[k][1] = t.y, xv[k][2] = t.z, xv[k][3] = t.w;
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) xv[k][j] = rel + j < valid ? x[e0 + rel + j] : 0.0f;
        }
    }
    const int64_t b0 = e0 / B;
    const auto store = [&](int k, const uint32_t q[4]) {
        // a block is written whole (padding codes are 0) if any of its elements is inside the array
        const int first = (k * kSub + 4 * lane) / B * B;
        if (FULL || first < valid) store_codes4<C, true>(codes, e0 + k * kSub + 4 * lane, q);
    };
    if constexpr (C == UF8) {
        uint32_t am = 0u;
#pragma unroll
        for (int k = 0; k < K; ++k) {
#pragma unroll
            for (int j = 0; j < 4; ++j) am = OpMax::f(am, abs_bits(xv[k][j]));
            if ((k + 1) % SUBS != 0) continue;
            am = group_reduce<OpMax, GL>(am);
            const int b = (k * kSub + (B < kSub ? 4 * lane : 0)) / B;
            const double r = am != 0u ? rdiv127((double)u2f(am)) : 0.0;
            if (lane % GL == 0 && (FULL || b * B < valid)) meta[b0 + b] = u2f(am);
#pragma unroll
            for (int s = k + 1 - SUBS; s <= k; ++s) {
                uint32_t q[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) q[j] = rint_low_bits((double)xv[s][j] * r) & 0xFFu;
                store(s, q);
            }
            am = 0u;
        }
    } else {
        constexpr int LEVELS = levels_of<C>();
        // 1. exact positive minimum and maximum of each block; lanes 2b, 2b + 1 take block b's
        const int pb = lane >> 1;
        uint32_t kmin = 0xFFFFFFFFu, kmax = 0u, mn = 0xFFFFFFFFu, mx = 0u;
#pragma unroll
        for (int k = 0; k < K; ++k) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                mn = OpMin::f(mn, pos_min_key(xv[k][j]));
                mx = OpMax::f(mx, pos_max_key(xv[k][j]));
            }
            if ((k + 1) % SUBS != 0) continue;
            mn = group_reduce<OpMin, GL>(mn);
            mx = group_reduce<OpMax, GL>(mx);
            if constexpr (B < kSub) {
                if (lane % GL == 0) skey[k * PER + lane / GL] = make_uint2(mn, mx);
            } else {
                kmin = pb == k / SUBS ? mn : kmin;
                kmax = pb == k / SUBS ? mx : kmax;
            }
            mn = 0xFFFFFFFFu;
            mx = 0u;
        }
        if constexpr (B < kSub) {
            __builtin_amdgcn_wave_barrier();  // this wavefront's LDS accesses run in order
            if (pb < NB) {
                kmin = skey[pb].x;
                kmax = skey[pb].y;
            }
        }
        // 2. the intervals, one block per lane pair (each lane one endpoint's logarithm)
        const bool any = kmax != 0u;
        const double lg = fit_log2(any ? u2f((lane & 1) ? kmax : kmin) : 1.0f);
        const double lg_other = dpp_d<kDppQuadXor1>(lg);
        const double lo = (lane & 1) ? lg_other : lg, hi = (lane & 1) ? lg : lg_other;
        const double l0 = lo > (double)log_floor ? lo : (double)log_floor;
        double l1 = hi < 126.0 ? hi : 126.0;
        if (kmin == kmax) l1 = l0 + 1.0;
        double dl = l1 - l0;
        dl = dl < 1e-12 ? 1e-12 : dl;
        if ((lane & 1) == 0 && pb < NB && (FULL || pb * B < valid)) {
            meta[2 * (b0 + pb)] = any ? (float)l0 : 0.0f;
            meta[2 * (b0 + pb) + 1] = any ? (float)dl : 0.0f;
        }
        const double inv = any ? (double)LEVELS / dl : 1.0;
        if constexpr (B < kSub) {
            if ((lane & 1) == 0 && pb < NB) senc[pb].e = al_enc_params(any ? l0 : 0.0, inv);
            __builtin_amdgcn_wave_barrier();
        }
        // 3. codes
        ALEnc enc;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            if constexpr (B < kSub)
                enc = senc[(k * kSub + 4 * lane) / B].e;
            else if (k % SUBS == 0)
                enc = al_enc_params(readlane_d(any ? l0 : 0.0, 2 * (k / SUBS)), readlane_d(inv, 2 * (k / SUBS)));
            uint32_t q[4];
#pragma unroll
            for (int j = 0; j < 4; ++j)
                q[j] = C == AL8 ? al_encode_f32(xv[k][j], enc) : al_encode_fast<LEVELS>(xv[k][j], enc);
            store(k, q);
        }
    }
}

__device__ __forceinline__ int64_t codec_chunk() {
    return xcd_order(blockIdx.x, gridDim.x) * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
}

// Loads. UF8 and AL16 codes are decoded with plain loads: a state that the last-level cache holds is read from it
// (20M values, UF8 18.3 us non-temporal, 15.8 plain; AL16 25.8 and 23.2; 300M no difference). UF8 encodes with
// plain loads while the input fits that cache (kCodecCached: 20M 17.6 and 16.2 us, 40M 33.8 and 29.1, but 100M 80 and 87); the
// other codes' arithmetic bounds them.
// Four waves per SIMD in both directions: the registers allow 7-8, but the streams mix less (50M values AL8
// B2048 -> fp32 -> AL16 B128: 109 us at 7-8, 107 at 4, 110 at 3, 125 at 2).
template <int C, int B, int K, bool NT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4, 4))) void quantize_kernel(const float* __restrict__ x, int64_t n, int64_t base,
                                                        float log_floor, void* codes, float* meta) {
    constexpr int E = 256 * K;
    constexpr int NS = C != UF8 && B < kSub ? E / B : 1;
    __shared__ uint2 skey[4][NS];
    __shared__ BlockEnc senc[4][NS];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t e0 = (base + codec_chunk()) * E, left = n - e0;
    const gp<const float> xg = to_g(x);
    const gp<uint8_t> cg = (gp<uint8_t>)to_g(codes);
    if (left >= E)
        quantize_chunk<C, B, K, NT, true>(xg, e0, E, lane, log_floor, cg, to_g(meta), skey[w], senc[w]);
    else if (left > 0)
        quantize_chunk<C, B, K, NT, false>(xg, e0, (int)left, lane, log_floor, cg, to_g(meta), skey[w], senc[w]);
}

// AL8 blocks of 512 and more decode through a table of the block's levels in LDS
// (255 evaluations, 4 per lane, in place of one per element; entry 0 is exact zero,
// so the values are those of al_decode_fast); other codes evaluate each element.
template <int C, int B, int K, bool FULL>
__device__ __forceinline__ void dequantize_chunk(gp<const uint8_t> codes, gp<const float> meta, int64_t e0, int valid,
                                                 int lane, gp<float> out, float* lut) {
    constexpr int NB = 256 * K / B;
    constexpr int SUBS = B < kSub ? 1 : B / kSub;
    constexpr bool LUT = C == AL8 && B >= 512;
    using W = typename std::conditional<C == AL16, uint2, uint32_t>::type;
    W w[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        const int rel = k * kSub + 4 * lane;
        if constexpr (FULL) {
            if constexpr (C == AL16)
                w[k] = ld_u2<false>(g_as<const void>(codes + 2 * (e0 + rel)));
            else
                w[k] = ld_u1<C == AL8>(g_as<const void>(codes + e0 + rel));
        } else {  // only the codes of the n elements are read
            uint32_t q[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                q[j] = 0u;
                if (rel + j < valid) q[j] = C == AL16 ? g_as<const uint16_t>(codes)[e0 + rel + j] : codes[e0 + rel + j];
            }
            if constexpr (C == AL16)
                w[k] = make_uint2(q[0] | (q[1] << 16), q[2] | (q[3] << 16));
            else
                w[k] = q[0] | (q[1] << 8) | (q[2] << 16) | (q[3] << 24);
        }
    }
    // decode step and l_min of block `lane`
    const int64_t b0 = e0 / B;
    float l32 = 0.0f;
    double step = 0.0;
    if (lane < NB && (FULL || lane * B < valid)) {
        if constexpr (C == UF8) {
            step = div127((double)meta[b0 + lane]);
        } else {
            l32 = meta[2 * (b0 + lane)];
            step = (double)meta[2 * (b0 + lane) + 1] / (double)levels_of<C>();
        }
    }
    if constexpr (LUT) {
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const double st = readlane_d(step, b), l = (double)u2f(readlane_u(f2u(l32), b));
#pragma unroll
            for (int i = 0; i < 4; ++i) lut[b * 256 + lane + 64 * i] = al_decode_fast((uint32_t)(lane + 64 * i), l, st, kExp2Codec);
        }
        __builtin_amdgcn_wave_barrier();  // this wavefront's LDS accesses run in order
    }
#pragma unroll
    for (int k = 0; k < K; ++k) {
        uint32_t q[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if constexpr (C == AL16)
                q[j] = ((j < 2 ? w[k].x : w[k].y) >> (16 * (j & 1))) & 0xFFFFu;
            else
                q[j] = (w[k] >> (8 * j)) & 0xFFu;
        }
        float o[4];
        if constexpr (LUT) {
#pragma unroll
            for (int j = 0; j < 4; ++j) o[j] = lut[(k / SUBS) * 256 + q[j]];
        } else {
            double st, l = 0.0;
            if constexpr (B >= kSub) {
                st = readlane_d(step, k / SUBS);
                if constexpr (C != UF8) l = (double)u2f(readlane_u(f2u(l32), k / SUBS));
            } else {
                const int src = (k * kSub + 4 * lane) / B;
                st = shfl_d(step, src);
                if constexpr (C != UF8) l = (double)__shfl(l32, src);
            }
#pragma unroll
            for (int j = 0; j < 4; ++j)
                o[j] = C == UF8 ? uf8_decode((int32_t)(int8_t)(uint8_t)q[j], st) : al_decode_fast(q[j], l, st, kExp2Codec);
        }
        const int rel = k * kSub + 4 * lane;
        if constexpr (FULL) {
            st_f4<false>(out + e0 + rel, make_float4(o[0], o[1], o[2], o[3]));
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (rel + j < valid) out[e0 + rel + j] = o[j];
        }
    }
}

template <int C, int B, int K>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4, 4))) void dequantize_kernel(const void* __restrict__ codes,
                                                          const float* __restrict__ meta, int64_t n, int64_t base,
                                                          float* __restrict__ out) {
    constexpr int E = 256 * K;
    __shared__ float lut[4][C == AL8 && B >= 512 ? E / B * 256 : 1];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t e0 = (base + codec_chunk()) * E, left = n - e0;
    const gp<const uint8_t> cg = (gp<const uint8_t>)to_g(codes);
    if (left >= E)
        dequantize_chunk<C, B, K, true>(cg, to_g(meta), e0, E, lane, to_g(out), lut[w]);
    else if (left > 0)
        dequantize_chunk<C, B, K, false>(cg, to_g(meta), e0, (int)left, lane, to_g(out), lut[w]);
}

// Device math primitives the codes rely on, evaluated elementwise so a test
// can compare them with the host: 0 = hardware fp32 log2, 1 = the binary64
// exp2 polynomial, 2 = binary64 log2, 3 = binary64 sqrt, 4 = 1 / sqrt(x),
// 5 / 6 = the UF8 quotients, 7 = the clipped-update quotient, 8 = the block
// endpoint log2 of an fp32 value, 9 = the clipped update of the CAME passes
// with 1 / clip folded into the row factor: fl32(fl64(fl64(r c) x) / d) for
// r, c, d below, eight consecutive inputs per decision as in the kernels (n a
// multiple of 8), 10 = the same for bf16 inputs (x a bf16 value) with r = d = 1
// and c = 0x1.00008c3a4f91dp7 (about 2^7 (1 + 2^-17)), just above the factor at which the CAME residual
// pass drops the range test: the midpoint test alone.
constexpr double kDiagR = 0.7310585786300049, kDiagC = 1234.5678901234567, kDiagD = 3.0000000000000004;
__global__ __launch_bounds__(256) void diag_math_kernel(int fn, const double* __restrict__ x, int64_t n,
                                                         double* __restrict__ out, const Exp2Coef cf) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    if (fn == 10) {
        constexpr double c = 0x1.00008c3a4f91dp7;  // r * c / d with r = d = 1: the row-safe threshold holds
        static_assert(c >= 0x1.00004p7, "above the row-safe factor");
        for (int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; 8 * g + 8 <= n; g += stride) {
            double q[8];
            float f[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) q[j] = (1.0 * c) * x[8 * g + j];
            if (!f32_midpoints_decided<8>(q, f)) {
#pragma unroll
                for (int j = 0; j < 8; ++j) f[j] = (float)(((1.0 * c) * x[8 * g + j]) / 1.0);
            }
#pragma unroll
            for (int j = 0; j < 8; ++j) out[8 * g + j] = (double)f[j];
        }
        return;
    }
    if (fn == 9) {
        const double rk = kDiagR * (1.0 / kDiagD);
        for (int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; 8 * g + 8 <= n; g += stride) {
            double q[8];
            float f[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) q[j] = (rk * kDiagC) * x[8 * g + j];
            if (!f32_roundings_decided<8>(q, f)) {
#pragma unroll
                for (int j = 0; j < 8; ++j) f[j] = (float)(((kDiagR * kDiagC) * x[8 * g + j]) / kDiagD);
            }
#pragma unroll
            for (int j = 0; j < 8; ++j) out[8 * g + j] = (double)f[j];
        }
        return;
    }
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        const double v = x[i];
        double r = 0.0;
        switch (fn) {
            case 0: r = (double)__builtin_amdgcn_logf((float)v); break;
            case 1: r = exp2_d(v, cf); break;
            case 2: r = log2(v); break;
            case 3: r = sqrt(v); break;
            case 4: r = 1.0 / sqrt(v); break;
            case 5: r = div127(v); break;
            case 6: r = rdiv127(v); break;
            case 7: r = (double)div_to_f32(v, 3.0, 1.0 / 3.0); break;
            case 8: r = fit_log2((float)v); break;
        }
        out[i] = r;
    }
}

hipError_t launch_diag_math(int fn, const double* x, int64_t n, double* out, int grid_cap, hipStream_t s) {
    const int64_t want = (n + 255) / 256;
    const int grid = (int)(want < grid_cap ? want : grid_cap);
    if (grid <= 0) return hipSuccess;
    hipLaunchKernelGGL(diag_math_kernel, dim3(grid), dim3(256), 0, s, fn, x, n, out, exp2_coef());
    return hipGetLastError();
}

// Sums of squares for the relative update error (section 3.2, Eq.
// update_error): out[0] = sum (a_i - b_i)^2, out[1] = sum b_i^2 over binary64
// terms, double-double partials per workgroup (fixed count and order), then
// one workgroup merges them; out[2 ..] holds the partials.
__global__ __launch_bounds__(256) void diff_norms_partial_kernel(const float* __restrict__ a,
                                                                 const float* __restrict__ b, int64_t n,
                                                                 double* __restrict__ part) {
    __shared__ DD sh[2][4];
    DD s0{0.0, 0.0}, s1{0.0, 0.0};
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        const double bi = (double)b[i];
        const double d = (double)a[i] - bi;
        dd_add(s0, d * d);
        dd_add(s1, bi * bi);
    }
    s0 = dd_wave_sum(s0);
    s1 = dd_wave_sum(s1);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if (lane == 0) {
        sh[0][w] = s0;
        sh[1][w] = s1;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        DD t0 = sh[0][0], t1 = sh[1][0];
        for (int k = 1; k < 4; ++k) {
            t0 = dd_merge(t0, sh[0][k]);
            t1 = dd_merge(t1, sh[1][k]);
        }
        double* o = part + 4 * blockIdx.x;
        o[0] = t0.hi;
        o[1] = t0.lo;
        o[2] = t1.hi;
        o[3] = t1.lo;
    }
}

__global__ __launch_bounds__(64) void diff_norms_final_kernel(const double* __restrict__ part, int np,
                                                              double* __restrict__ out) {
    DD s0{0.0, 0.0}, s1{0.0, 0.0};
    for (int k = threadIdx.x; k < np; k += 64) {
        s0 = dd_merge(s0, DD{part[4 * k], part[4 * k + 1]});
        s1 = dd_merge(s1, DD{part[4 * k + 2], part[4 * k + 3]});
    }
    s0 = dd_wave_sum(s0);
    s1 = dd_wave_sum(s1);
    if (threadIdx.x == 0) {
        out[0] = dd_value(s0);
        out[1] = dd_value(s1);
    }
}

hipError_t launch_diff_norms(const float* a, const float* b, int64_t n, double* out, hipStream_t s) {
    constexpr int kParts = kDiffNormParts;
    const int64_t want = (n + 255) / 256;
    const int np = (int)(want < kParts ? (want > 0 ? want : 1) : kParts);
    hipLaunchKernelGGL(diff_norms_partial_kernel, dim3(np), dim3(256), 0, s, a, b, n, out + 2);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(diff_norms_final_kernel, dim3(1), dim3(64), 0, s, out + 2, np, out);
    return hipGetLastError();
}

// Streaming ceiling of the fused AdamW access pattern: per element read p
// (fp32), g (bf16), m and v (1 byte each), write p, m, v -- the same bytes,
// lane mapping and launch shape as the AdamW kernel at B_V 2048 (one 2048-element chunk
// per wavefront in two load phases of four 256-element sub-tiles, 4
// consecutive elements per lane, XCD-contiguous workgroup order; smaller blocks take
// chunks of 512 or 1024 in one phase but in long lists), with no
// optimizer arithmetic. NT selects non-temporal loads and stores.
template <bool NT>
__global__ __launch_bounds__(256) void stream_kernel(float* __restrict__ p, const uint16_t* __restrict__ g,
                                                      uint8_t* __restrict__ m, uint8_t* __restrict__ v,
                                                      int64_t chunk_base, int64_t chunks) {
    const int lane = threadIdx.x & 63;
    const int64_t c = chunk_base + xcd_order(blockIdx.x, gridDim.x) * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (c >= chunks) return;
#pragma unroll
    for (int ph = 0; ph < 2; ++ph) {
        if (ph > 0) __builtin_amdgcn_sched_barrier(0);
        float4 pv[4];
        uint2 gv[4];
        uint32_t mv[4], vv[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int64_t e = c * 2048 + (ph * 4 + k) * 256 + 4 * lane;
            pv[k] = ld_f4<NT>(p + e);
            gv[k] = ld_u2<NT>(g + e);
            mv[k] = ld_u1<NT>(m + e);
            vv[k] = ld_u1<NT>(v + e);
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int64_t e = c * 2048 + (ph * 4 + k) * 256 + 4 * lane;
            float4 o = pv[k];
            o.x += bf16_to_f32(gv[k].x & 0xFFFFu);
            o.w += bf16_to_f32(gv[k].y >> 16);
            st_f4<NT>(p + e, o);
            st_u1<NT>(m + e, mv[k] ^ vv[k]);
            st_u1<NT>(v + e, vv[k] + 0x01010101u);
        }
    }
}

// Best streaming shape found for the same byte mix (a reference rate, not
// the step's layout): one 4096-element chunk per wavefront, every stream read
// 16 bytes per lane (p: 4 elements, g: 8, m and v: 16 per lane), all loads of
// the chunk issued before any store, XCD-contiguous order. Writes p + 1,
// m ^ v, v + 1 (per byte); g is read and discarded.
__global__ __launch_bounds__(256) void stream_wide_kernel(float* __restrict__ p, const uint16_t* __restrict__ g,
                                                          uint8_t* __restrict__ m, uint8_t* __restrict__ v,
                                                          int64_t chunk_base, int64_t chunks) {
    typedef uint32_t u4 __attribute__((ext_vector_type(4)));
    const int lane = threadIdx.x & 63;
    const int64_t c = chunk_base + xcd_order(blockIdx.x, gridDim.x) * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (c >= chunks) return;
    const int64_t e0 = c * 4096;
    nt_f4 pv[16];
    u4 gv[8], mv[4], vv[4];
#pragma unroll
    for (int i = 0; i < 16; ++i) pv[i] = __builtin_nontemporal_load(reinterpret_cast<const nt_f4*>(p + e0 + i * 256 + 4 * lane));
#pragma unroll
    for (int i = 0; i < 8; ++i) gv[i] = __builtin_nontemporal_load(reinterpret_cast<const u4*>(g + e0 + i * 512 + 8 * lane));
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        mv[i] = __builtin_nontemporal_load(reinterpret_cast<const u4*>(m + e0 + i * 1024 + 16 * lane));
        vv[i] = __builtin_nontemporal_load(reinterpret_cast<const u4*>(v + e0 + i * 1024 + 16 * lane));
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) asm volatile("" ::"v"(gv[i]));  // the gradient bytes are read, not used
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < 16; ++i)
        __builtin_nontemporal_store(pv[i] + 1.0f, reinterpret_cast<nt_f4*>(p + e0 + i * 256 + 4 * lane));
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        __builtin_nontemporal_store(mv[i] ^ vv[i], reinterpret_cast<u4*>(m + e0 + i * 1024 + 16 * lane));
        __builtin_nontemporal_store(vv[i] + 0x01010101u, reinterpret_cast<u4*>(v + e0 + i * 1024 + 16 * lane));
    }
}

hipError_t launch_diag_stream(int mode, float* p, const uint16_t* g, uint8_t* m, uint8_t* v, int64_t n,
                              hipStream_t s) {
    const bool wide = (mode & 2) != 0;
    const int64_t chunks = n / (wide ? 4096 : 2048);
    constexpr int64_t kMaxGrid = int64_t(1) << 30;
    for (int64_t base = 0; base < chunks; base += 4 * kMaxGrid) {
        const int64_t left = (chunks - base + 3) / 4;
        const int64_t grid = left < kMaxGrid ? left : kMaxGrid;
        if (wide)
            hipLaunchKernelGGL(stream_wide_kernel, dim3((unsigned)grid), dim3(256), 0, s, p, g, m, v, base, chunks);
        else if (mode & 1)
            hipLaunchKernelGGL(stream_kernel<true>, dim3((unsigned)grid), dim3(256), 0, s, p, g, m, v, base, chunks);
        else
            hipLaunchKernelGGL(stream_kernel<false>, dim3((unsigned)grid), dim3(256), 0, s, p, g, m, v, base, chunks);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// Chunks of 2048 elements (K = 8), or of max(B, 256) where the array has too few
// of those to give every SIMD a wavefront: below 2^21 elements. AL16's arithmetic per element wants more wavefronts
// for longer: short chunks are faster up to about 4M elements encoding (us at 2.2M and 4M with long and short ones: B 128
// 10.8 and 8.1, 11.4 and 12.3; B 1024 9.6 and 7.7, 10.5 and 9.6), 7M decoding (5M and 8M: B 128 8.9 and 8.5, 12.1 and
// 12.9; B 512 8.5 and 7.5, 11.6 and 10.4). AL8 at 4M: encoding 7.2 and 8.7, decoding 7.0 and 7.7.
constexpr int64_t codec_long(int c, bool encode) {
    return c == AL16 ? (encode ? int64_t(1) << 22 : int64_t(7) << 20) : int64_t(1) << 21;
}
constexpr int64_t kCodecCached = int64_t(1) << 26;  // 256 MB of fp32

// One wavefront per chunk, 4 per workgroup; launches beyond 2^32 chunks are split.
template <class F>
static hipError_t codec_launch(int64_t n, int64_t elems, F launch) {
    constexpr int64_t kMaxGrid = int64_t(1) << 30;
    const int64_t chunks = (n + elems - 1) / elems;
    for (int64_t base = 0; base < chunks; base += 4 * kMaxGrid) {
        const int64_t left = (chunks - base + 3) / 4;
        launch(dim3((unsigned)(left < kMaxGrid ? left : kMaxGrid)), base);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template <int C, int B, int K, bool NT>
static hipError_t quant_k(const float* x, int64_t n, float lf, void* codes, float* meta, hipStream_t s) {
    return codec_launch(n, K * kSub, [&](dim3 g, int64_t base) {
        hipLaunchKernelGGL((quantize_kernel<C, B, K, NT>), g, dim3(256), 0, s, x, n, base, lf, codes, meta);
    });
}

template <int C, int B>
static hipError_t quant_t(const float* x, int64_t n, float lf, void* codes, float* meta, hipStream_t s) {
    constexpr int KS = B > kSub ? B / kSub : 1;
    constexpr bool NT = C != UF8;
    if (n < codec_long(C, true)) return quant_k<C, B, KS, NT>(x, n, lf, codes, meta, s);
    if (n < kCodecCached) return quant_k<C, B, 8, NT>(x, n, lf, codes, meta, s);
    return quant_k<C, B, 8, true>(x, n, lf, codes, meta, s);
}

template <int C, int B>
static hipError_t dequant_t(const void* codes, const float* meta, int64_t n, float* out, hipStream_t s) {
    constexpr int KS = B > kSub ? B / kSub : 1;
    if (n >= codec_long(C, false))
        return codec_launch(n, 2048, [&](dim3 g, int64_t base) {
            hipLaunchKernelGGL((dequantize_kernel<C, B, 8>), g, dim3(256), 0, s, codes, meta, n, base, out);
        });
    return codec_launch(n, KS * kSub, [&](dim3 g, int64_t base) {
        hipLaunchKernelGGL((dequantize_kernel<C, B, KS>), g, dim3(256), 0, s, codes, meta, n, base, out);
    });
}

#define AL_BLOCKS(F, ...)                       \
    switch (block) {                            \
        case 64: return F<C, 64>(__VA_ARGS__);     \
        case 128: return F<C, 128>(__VA_ARGS__);   \
        case 256: return F<C, 256>(__VA_ARGS__);   \
        case 512: return F<C, 512>(__VA_ARGS__);   \
        case 1024: return F<C, 1024>(__VA_ARGS__); \
        case 2048: return F<C, 2048>(__VA_ARGS__); \
    }                                           \
    return hipErrorInvalidValue;

template <int C>
static hipError_t quant_b(const float* x, int64_t n, int block, float lf, void* codes, float* meta, hipStream_t s) {
    AL_BLOCKS(quant_t, x, n, lf, codes, meta, s)
}

template <int C>
static hipError_t dequant_b(const void* codes, const float* meta, int64_t n, int block, float* out, hipStream_t s) {
    AL_BLOCKS(dequant_t, codes, meta, n, out, s)
}
#undef AL_BLOCKS

hipError_t launch_quantize(int codec, const float* x, int64_t n, int block, float log_floor, void* codes,
                           float* meta, hipStream_t s) {
    switch (codec) {
        case AL8: return quant_b<AL8>(x, n, block, log_floor, codes, meta, s);
        case AL16: return quant_b<AL16>(x, n, block, log_floor, codes, meta, s);
        case UF8: return quant_b<UF8>(x, n, block, log_floor, codes, meta, s);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_dequantize(int codec, const void* codes, const float* meta, int64_t n, int block, float* out,
                             hipStream_t s) {
    switch (codec) {
        case AL8: return dequant_b<AL8>(codes, meta, n, block, out, s);
        case AL16: return dequant_b<AL16>(codes, meta, n, block, out, s);
        case UF8: return dequant_b<UF8>(codes, meta, n, block, out, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace al
