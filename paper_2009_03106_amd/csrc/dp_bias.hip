// Parameters whose per-example gradients are column sums, small enough ([B, d] floats) to
// materialise: bias vectors, u_i = sum_t G_i[t, :] (dL/db = dL/dz for a fully-connected
// layer, Section 5.1; summed over the positions that share the bias, Section 5.3), and
// LayerNorm scale / shift, sum_t G_i[t, :] (*) Hbar_i[t, :] and sum_t G_i[t, :] (Section 5.5,
// Algorithm 5); their squared norms; and the clipped sum  sum_i nu_i u_i.
// All of it is bandwidth-bound; every sum runs in a fixed order (no atomics).
#include <algorithm>
#include "dp_common.h"
#include "dp_internal.h"
#include "dp_noise.h"
#include <type_traits>

namespace dpk {

namespace {

// One workgroup per (example, chunk of columns).  The 256 threads form rg row groups x ct column
// threads (ct = 1 << ctl); a thread owns VEC consecutive columns (one 16-byte load per row) and
// adds rows rgid, rgid + rg, ... in ascending order; the rg partial sums are then added in the
// order 0 .. rg-1.  Needs D % VEC == 0 (with the 16-byte aligned base every load is aligned).
// PROD: a second input Hb of the same shape; u2 gets the plain column sums and u the sums of G (*) Hb.
// DT (type of G), DTH (type of Hb): 0 = float32, 1 = bf16, 2 = fp16, 3 = e4m3, 4 = e5m2; both of the same width
template <int DT> struct ElemBytes { static constexpr int value = DT == 0 ? 4 : (DT >= 3 ? 1 : 2); };
// one 8-bit float -> float32 (e5m2 is the upper byte of an fp16)
template <int DT> __device__ __forceinline__ float f8_byte(uint32_t word, int which) {
    if (DT == 4) return (float)__builtin_bit_cast(_Float16, (uint16_t)(((word >> (8 * which)) & 0xffu) << 8));
    return which == 0 ? __builtin_amdgcn_cvt_f32_fp8((int)word, 0) : which == 1 ? __builtin_amdgcn_cvt_f32_fp8((int)word, 1)
         : which == 2 ? __builtin_amdgcn_cvt_f32_fp8((int)word, 2) : __builtin_amdgcn_cvt_f32_fp8((int)word, 3);
}
template <int DT, bool PROD, int DTH = DT>
__device__ __forceinline__ void bias_rows_block(const void* __restrict__ G, const void* __restrict__ Hb, int T, int D, int ctl,
                                                float* __restrict__ u, float* __restrict__ u2, int bx, int ex, float* sqnorm = nullptr, int accumulate = 0) {
    constexpr int ES = ElemBytes<DT>::value;          // bytes per element
    static_assert(ElemBytes<DTH>::value == ES, "G and Hb of one width");
    constexpr int VEC = 16 / ES;
    __shared__ float part[kThreads][PROD ? 2 * VEC : VEC];
    const int tid = threadIdx.x, ct = 1 << ctl, rg = kThreads >> ctl;
    const int ctid = tid & (ct - 1), rgid = tid >> ctl;
    const int col0 = (bx * ct + ctid) * VEC;
    float acc[VEC], acc2[VEC];                        // acc2 (PROD only): plain sums
#pragma unroll
    for (int v = 0; v < VEC; ++v) { acc[v] = 0.f; acc2[v] = 0.f; }
    auto widen = [&](const uint4& w, float (&x)[VEC], auto tag) {
        constexpr int E = decltype(tag)::value;
        const uint32_t d[4] = {w.x, w.y, w.z, w.w};
        if constexpr (E >= 3) {
            // two conversions per instruction (v_cvt_pk_f32_fp8 / _bf8: the low or the high 16 bits of the word)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                f32x2 lo, hi;
                if constexpr (E == 3) { lo = __builtin_amdgcn_cvt_pk_f32_fp8((int)d[j], false); hi = __builtin_amdgcn_cvt_pk_f32_fp8((int)d[j], true); }
                else                  { lo = __builtin_amdgcn_cvt_pk_f32_bf8((int)d[j], false); hi = __builtin_amdgcn_cvt_pk_f32_bf8((int)d[j], true); }
                x[4 * j] = lo[0]; x[4 * j + 1] = lo[1]; x[4 * j + 2] = hi[0]; x[4 * j + 3] = hi[1];
            }
        } else if constexpr (E != 0) {
#pragma unroll
            for (int j = 0; j < 4; ++j) { x[2 * j] = In16<E == 2>::lo(d[j]); x[2 * j + 1] = In16<E == 2>::hi(d[j]); }
        } else {
            x[0] = __uint_as_float(w.x); x[1] = __uint_as_float(w.y); x[2] = __uint_as_float(w.z); x[3] = __uint_as_float(w.w);
        }
    };
    auto add = [&](const uint4& w) {
        float x[VEC];
        widen(w, x, std::integral_constant<int, DT>{});
#pragma unroll
        for (int v = 0; v < VEC; ++v) acc[v] += x[v];
    };
    auto add_prod = [&](const uint4& w, const uint4& h) {
        float x[VEC], y[VEC];
        widen(w, x, std::integral_constant<int, DT>{});
        widen(h, y, std::integral_constant<int, DTH>{});
#pragma unroll
        for (int v = 0; v < VEC; ++v) { acc[v] += x[v] * y[v]; acc2[v] += x[v]; }
    };
    if (col0 < D) {
        const size_t row_bytes = (size_t)D * ES;
        const unsigned char* p = static_cast<const unsigned char*>(G) + ((size_t)ex * T) * row_bytes + (size_t)col0 * ES;
        int t = rgid;
        if (PROD) {
            const unsigned char* q = static_cast<const unsigned char*>(Hb) + ((size_t)ex * T) * row_bytes + (size_t)col0 * ES;
            for (; t + 3 * rg < T; t += 4 * rg) {      // eight loads in flight, added in row order
                uint4 w[4], h[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    w[k] = *reinterpret_cast<const uint4*>(p + (size_t)(t + k * rg) * row_bytes);
                    h[k] = *reinterpret_cast<const uint4*>(q + (size_t)(t + k * rg) * row_bytes);
                }
#pragma unroll
                for (int k = 0; k < 4; ++k) add_prod(w[k], h[k]);
            }
            for (; t < T; t += rg)
                add_prod(*reinterpret_cast<const uint4*>(p + (size_t)t * row_bytes), *reinterpret_cast<const uint4*>(q + (size_t)t * row_bytes));
        } else {
            for (; t + 7 * rg < T; t += 8 * rg) {      // eight loads in flight, added in row order
                uint4 w[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) w[k] = *reinterpret_cast<const uint4*>(p + (size_t)(t + k * rg) * row_bytes);
#pragma unroll
                for (int k = 0; k < 8; ++k) add(w[k]);
            }
            for (; t < T; t += rg) add(*reinterpret_cast<const uint4*>(p + (size_t)t * row_bytes));
        }
    }
#pragma unroll
    for (int v = 0; v < VEC; ++v) { part[tid][v] = acc[v]; if (PROD) part[tid][VEC + v] = acc2[v]; }
    __syncthreads();
    if (rgid == 0 && col0 < D) {
        for (int r = 1; r < rg; ++r)
#pragma unroll
            for (int v = 0; v < VEC; ++v) { acc[v] += part[r * ct + ctid][v]; if (PROD) acc2[v] += part[r * ct + ctid][VEC + v]; }
        float* o = u + (size_t)ex * D + col0;
#pragma unroll
        for (int v = 0; v < VEC; ++v) o[v] = acc[v];
        if (PROD) {
            float* o2 = u2 + (size_t)ex * D + col0;
#pragma unroll
            for (int v = 0; v < VEC; ++v) o2[v] = acc2[v];
        }
    }
    if (sqnorm && tid < kWave) {                       // the workgroup has the whole rows (ct <= 64 threads of the first wave)
        float s = 0.f;
        if (rgid == 0 && col0 < D) {
#pragma unroll
            for (int v = 0; v < VEC; ++v) s += PROD ? acc[v] * acc[v] + acc2[v] * acc2[v] : acc[v] * acc[v];
        }
        s = wave_sum(s);
        if (tid == 0) sqnorm[ex] = accumulate ? sqnorm[ex] + s : s;
    }
}

template <int DT, bool PROD, int DTH = DT>
__global__ __launch_bounds__(kThreads) void k_bias_rows(const void* __restrict__ G, const void* __restrict__ Hb, int T, int D, int ctl,
                                                        float* __restrict__ u, float* __restrict__ u2, float* __restrict__ sqnorm, int accumulate) {
    bias_rows_block<DT, PROD, DTH>(G, Hb, T, D, ctl, u, u2, blockIdx.x, blockIdx.y, sqnorm, accumulate);
}

// Any D: 32 columns a workgroup, its 8 row groups add rows g, g + 8, ... in ascending order, four loads in flight, and the
// groups' sums are added in their order.  (One thread per column, a load after the other: 15 examples of 447 x 940 took 120 us.)
template <int DT> __device__ __forceinline__ float load_elem(const void* p, size_t k) {
    if (DT >= 3) return f8_byte<DT>(static_cast<const unsigned char*>(p)[k], 0);
    if (DT != 0) return In16<DT == 2>::lo(static_cast<const uint16_t*>(p)[k]);
    return static_cast<const float*>(p)[k];
}
constexpr int kScalarColumns = 32;
template <int DT, bool PROD, int DTH = DT>
__device__ __forceinline__ void bias_rows_scalar_block(const void* __restrict__ G, const void* __restrict__ Hb, int T, int D,
                                                       float* __restrict__ u, float* __restrict__ u2, int bx, int ex) {
    constexpr int RG = kThreads / kScalarColumns;
    __shared__ float part[PROD ? 2 : 1][RG][kScalarColumns];
    const int cl = threadIdx.x & (kScalarColumns - 1), g = threadIdx.x / kScalarColumns;
    const int q = bx * kScalarColumns + cl;
    float acc = 0.f, acc2 = 0.f;
    if (q < D) {
        const size_t base = (size_t)ex * T * D + q;
        auto add = [&](float x, float h) {
            if (PROD) { acc += x * h; acc2 += x; } else acc += x;
        };
        int t = g;
        for (; t + 3 * RG < T; t += 4 * RG) {
            float x[4], h[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                x[k] = load_elem<DT>(G, base + (size_t)(t + k * RG) * D);
                h[k] = PROD ? load_elem<DTH>(Hb, base + (size_t)(t + k * RG) * D) : 0.f;
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) add(x[k], h[k]);
        }
        for (; t < T; t += RG) add(load_elem<DT>(G, base + (size_t)t * D), PROD ? load_elem<DTH>(Hb, base + (size_t)t * D) : 0.f);
    }
    part[0][g][cl] = acc;
    if (PROD) part[1][g][cl] = acc2;
    __syncthreads();
    if (g != 0 || q >= D) return;
#pragma unroll
    for (int r = 1; r < RG; ++r) { acc += part[0][r][cl]; if (PROD) acc2 += part[1][r][cl]; }
    u[(size_t)ex * D + q] = acc;
    if (PROD) u2[(size_t)ex * D + q] = acc2;
}
template <int DT, bool PROD, int DTH = DT>
__global__ __launch_bounds__(kThreads) void k_bias_rows_scalar(const void* __restrict__ G, const void* __restrict__ Hb, int T, int D,
                                                               float* __restrict__ u, float* __restrict__ u2) {
    bias_rows_scalar_block<DT, PROD, DTH>(G, Hb, T, D, u, u2, blockIdx.x, blockIdx.y);
}

// The bias rows of several layers in one launch, each with its own launch's split (ctl; < 0: 32 columns a workgroup): a
// layer of 32 examples is a few hundred workgroups of 5 to 6 us, five of them and their norms were ten launches.
struct BiasRowsLayers { const void* G[kBiasLayers]; float* u[kBiasLayers]; int T[kBiasLayers], D[kBiasLayers], ctl[kBiasLayers],
                        chunks[kBiasLayers], first_block[kBiasLayers]; int n_layers; };
template <int DT>
__global__ __launch_bounds__(kThreads) void k_bias_rows_layers(BiasRowsLayers a) {
    int l = 0;
    while (l + 1 < a.n_layers && (int)blockIdx.x >= a.first_block[l + 1]) ++l;
    const int b = blockIdx.x - a.first_block[l], ex = b / a.chunks[l], bx = b - ex * a.chunks[l];
    if (a.ctl[l] >= 0) bias_rows_block<DT, false>(a.G[l], nullptr, a.T[l], a.D[l], a.ctl[l], a.u[l], nullptr, bx, ex);
    else               bias_rows_scalar_block<DT, false>(a.G[l], nullptr, a.T[l], a.D[l], a.u[l], nullptr, bx, ex);
}

// s_i (+)= sum_q u[i, q]^2 (+ sum_q u2[i, q]^2 when u2 is given: LayerNorm's scale and shift rows in one launch):
// one wave per example, four per workgroup; lane l adds the 16-byte pieces l, l + 64, ... of the row (four loads in
// flight), then a shuffle tree.  The order of the additions is fixed.
__device__ __forceinline__ float row_sq(const float* __restrict__ p, int D, int lane) {
    float acc = 0.f;
    if ((D & 3) == 0 && (reinterpret_cast<uintptr_t>(p) & 15) == 0) {
        const float4* p4 = reinterpret_cast<const float4*>(p);
        const int n4 = D >> 2;
        int q = lane;
        for (; q + 3 * kWave < n4; q += 4 * kWave) {
            const float4 a = p4[q], b = p4[q + kWave], c = p4[q + 2 * kWave], d = p4[q + 3 * kWave];
            acc += a.x * a.x + a.y * a.y + a.z * a.z + a.w * a.w;
            acc += b.x * b.x + b.y * b.y + b.z * b.z + b.w * b.w;
            acc += c.x * c.x + c.y * c.y + c.z * c.z + c.w * c.w;
            acc += d.x * d.x + d.y * d.y + d.z * d.z + d.w * d.w;
        }
        for (; q < n4; q += kWave) { const float4 a = p4[q]; acc += a.x * a.x + a.y * a.y + a.z * a.z + a.w * a.w; }
    } else {
        int q = lane;
        for (; q + 7 * kWave < D; q += 8 * kWave) {      // eight loads in flight, added in order
            float v[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] = p[q + k * kWave];
#pragma unroll
            for (int k = 0; k < 8; ++k) acc += v[k] * v[k];
        }
        for (; q < D; q += kWave) { const float v = p[q]; acc += v * v; }
    }
    return wave_sum(acc);
}
__global__ __launch_bounds__(kThreads) void k_rows_sqnorm(const float* __restrict__ u, const float* __restrict__ u2, int B, int D,
                                                          int accumulate, float* __restrict__ sqnorm) {
    const int lane = threadIdx.x & (kWave - 1);
    const int ex = blockIdx.x * (kThreads / kWave) + (threadIdx.x >> 6);
    if (ex >= B) return;
    const float a = row_sq(u + (size_t)ex * D, D, lane);
    const float b = u2 ? row_sq(u2 + (size_t)ex * D, D, lane) : 0.f;
    if (lane == 0) {
        float s = accumulate ? sqnorm[ex] + a : a;
        if (u2) s += b;
        sqnorm[ex] = s;
    }
}

// the same for several layers' rows, added in the order given: the bits of one launch of k_rows_sqnorm per layer (a call for one
// layer whose launch has whole rows adds their squares by pieces: equal to float32 rounding).  A workgroup per example, its
// waves take the layers in turn (one wave for all of them: 14 us for five layers of 656 to 1968 columns)
struct RowsLayers { const float* u[kBiasLayers]; int D[kBiasLayers]; int n_layers; };
__global__ __launch_bounds__(kThreads) void k_rows_sqnorm_layers(RowsLayers a, int accumulate, float* __restrict__ sqnorm) {
    __shared__ float sums[kBiasLayers];
    const int lane = threadIdx.x & (kWave - 1), ex = blockIdx.x;
    for (int l = threadIdx.x >> 6; l < a.n_layers; l += kThreads / kWave) {
        const float v = row_sq(a.u[l] + (size_t)ex * a.D[l], a.D[l], lane);
        if (lane == 0) sums[l] = v;
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    float s = accumulate ? sqnorm[ex] + sums[0] : sums[0];
    for (int l = 1; l < a.n_layers; ++l) s += sums[l];
    sqnorm[ex] = s;
}

// grad_b[q] (+)= sum_i nu_i u[i, q].  A workgroup owns 32 columns; its NG row groups add examples g, g + NG, ... in
// ascending order (four loads in flight each), and the NG partial sums are added in the order g = 0 .. NG - 1: a
// fixed order, so the result is reproducible.  (One thread per column walking all B examples one dependent load
// after the other took 17 us for 256 examples.)  NG = 8 for small batches; 32 (1024 threads per workgroup) from
// 2048 examples on: the grid is only d_out / 32 workgroups, so a long batch needs the loads of many threads in
// flight per workgroup (B = 65536, d_out = 512: 0.70 ms with 8 groups).
template <int NG>
__device__ __forceinline__ void clipped_bias_block(const float* __restrict__ u, const float* __restrict__ clip, int B, int D,
                                                   int accumulate, float* __restrict__ grad_b, int bx, const NoiseArgs& nz) {
    __shared__ float part[NG][32];
    const int g = threadIdx.x >> 5, cl = threadIdx.x & 31;
    const int q = bx * 32 + cl;
    float acc = 0.f;
    if (q < D) {
        int i = g;
        for (; i + 3 * NG < B; i += 4 * NG) {
            const float v0 = u[(size_t)i * D + q], v1 = u[(size_t)(i + NG) * D + q];
            const float v2 = u[(size_t)(i + 2 * NG) * D + q], v3 = u[(size_t)(i + 3 * NG) * D + q];
            acc += clip[i] * v0; acc += clip[i + NG] * v1; acc += clip[i + 2 * NG] * v2; acc += clip[i + 3 * NG] * v3;
        }
        for (; i < B; i += NG) acc += clip[i] * u[(size_t)i * D + q];
    }
    part[g][cl] = acc;
    __syncthreads();
    if (g == 0 && q < D) {
#pragma unroll
        for (int k = 1; k < NG; ++k) acc += part[k][cl];
        float v = accumulate ? grad_b[q] + acc : acc;
        if (nz.stddev != 0.0f) {
            // entry q of the layer's stretch of the noise stream: slot (offset + q) % 4 of Philox block (offset + q) / 4
            const uint64_t j = nz.offset + (uint64_t)q;
            const U4 w = philox4x32_10((uint32_t)(j >> 2), (uint32_t)(j >> 34), 0u, 0u, nz.k0, nz.k1);
            float z0, z1;
            if (j & 2) box_muller(w.z, w.w, z0, z1); else box_muller(w.x, w.y, z0, z1);
            v += nz.stddev * ((j & 1) ? z1 : z0);
        }
        grad_b[q] = v;
    }
}
template <int NG>
__global__ __launch_bounds__(NG * 32) void k_clipped_bias(const float* __restrict__ u, const float* __restrict__ clip, int B, int D,
                                                          int accumulate, float* __restrict__ grad_b) {
    clipped_bias_block<NG>(u, clip, B, D, accumulate, grad_b, blockIdx.x, NoiseArgs{0.0f, 0u, 0u, 0u});
}
// several layers' bias gradients and their noise in one launch
struct ClippedBiasLayers { const float* u[kBiasLayers]; const float* clip[kBiasLayers]; float* grad_b[kBiasLayers];
                           uint64_t noise_offset[kBiasLayers]; int D[kBiasLayers], first_block[kBiasLayers]; int n_layers; };
template <int NG>
__global__ __launch_bounds__(NG * 32) void k_clipped_bias_layers(ClippedBiasLayers a, int B, int accumulate, NoiseArgs nz) {
    int l = 0;
    while (l + 1 < a.n_layers && (int)blockIdx.x >= a.first_block[l + 1]) ++l;
    nz.offset = a.noise_offset[l];
    clipped_bias_block<NG>(a.u[l], a.clip[l], B, a.D[l], accumulate, a.grad_b[l], blockIdx.x - a.first_block[l], nz);
}

// log2 of the column threads of k_bias_rows: next power of two, at most 64, but narrower column chunks (down to 16 threads =
// 256-byte row pieces) while the grid is too small to keep enough loads in flight for HBM
int column_threads_log2(int nvec, int B) {
    int ctl = 0;
    while (ctl < 6 && (1 << ctl) < nvec) ++ctl;
    while (ctl > 4 && (int64_t)((nvec + (1 << ctl) - 1) >> ctl) * B < 1024) --ctl;
    return ctl;
}
// whether a workgroup of k_bias_rows has an example's whole rows
bool bias_rows_whole(int B, int D, int vec) {
    return D % vec == 0 && (D / vec) <= (1 << column_threads_log2(D / vec, B));
}
template <int DT, int DTH = DT> void launch_bias_rows_dt(const void* G, const void* Hb, int B, int T, int D, float* u, float* u2, float* sqnorm, int accumulate, hipStream_t st) {
    constexpr int vec = 16 / ElemBytes<DT>::value;
    const bool prod = Hb != nullptr;
    if (D % vec == 0) {
        const int nvec = D / vec;
        const int ctl = column_threads_log2(nvec, B);
        const dim3 grid((unsigned)((nvec + (1 << ctl) - 1) >> ctl), (unsigned)B);
        if (prod) k_bias_rows<DT, true, DTH><<<grid, kThreads, 0, st>>>(G, Hb, T, D, ctl, u, u2, sqnorm, accumulate);
        else      k_bias_rows<DT, false><<<grid, kThreads, 0, st>>>(G, Hb, T, D, ctl, u, u2, sqnorm, accumulate);
    } else {
        const dim3 grid((unsigned)((D + kScalarColumns - 1) / kScalarColumns), (unsigned)B);
        if (prod) k_bias_rows_scalar<DT, true, DTH><<<grid, kThreads, 0, st>>>(G, Hb, T, D, u, u2);
        else      k_bias_rows_scalar<DT, false><<<grid, kThreads, 0, st>>>(G, Hb, T, D, u, u2);
    }
}

}  // namespace

// Hb == nullptr: u = column sums of G.  Otherwise u = column sums of G (*) Hb and u2 = column sums of G.  s_i (+)= the rows' sums of
// squares, by the same launch where a workgroup has whole rows.
// dt: type of G and Hb as above; 5: G e5m2 with Hb e4m3.
hipError_t launch_bias_rows(const void* G, const void* Hb, int B, int T, int D, int dt, float* u, float* u2, bool accumulate, float* sqnorm, hipStream_t st) {
    // the examples are the grid's y dimension (at most 65535), a launch has at most 2^24 workgroups: larger batches go in
    // several launches
    const int most = std::min(65535, ((1 << 24) - 1) / ceil_div(D, kScalarColumns));
    const size_t es = dt == 0 ? 4 : (dt >= 3 ? 1 : 2);
    for (int b0 = 0; b0 < B; b0 += most) {
        const int nb = std::min(B - b0, most);
        const size_t in_off = (size_t)b0 * T * D * es, out_off = (size_t)b0 * D;
        const void* g = static_cast<const unsigned char*>(G) + in_off;
        const void* h = Hb ? static_cast<const unsigned char*>(Hb) + in_off : nullptr;
        float* pu = u + out_off;
        float* pu2 = u2 ? u2 + out_off : nullptr;
        // (with rows in several pieces the norms take a launch of their own)
        float* sq = bias_rows_whole(nb, D, (int)(16 / es)) ? sqnorm + b0 : nullptr;
        if (dt == 5)      launch_bias_rows_dt<4, 3>(g, h, nb, T, D, pu, pu2, sq, accumulate ? 1 : 0, st);
        else if (dt == 4) launch_bias_rows_dt<4>(g, h, nb, T, D, pu, pu2, sq, accumulate ? 1 : 0, st);
        else if (dt == 3) launch_bias_rows_dt<3>(g, h, nb, T, D, pu, pu2, sq, accumulate ? 1 : 0, st);
        else if (dt == 2) launch_bias_rows_dt<2>(g, h, nb, T, D, pu, pu2, sq, accumulate ? 1 : 0, st);
        else if (dt == 1) launch_bias_rows_dt<1>(g, h, nb, T, D, pu, pu2, sq, accumulate ? 1 : 0, st);
        else              launch_bias_rows_dt<0>(g, h, nb, T, D, pu, pu2, sq, accumulate ? 1 : 0, st);
        hipError_t e = hipGetLastError();
        if (e == hipSuccess && !sq) e = launch_rows_sqnorm(pu, nb, D, accumulate, sqnorm + b0, st, pu2);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

// Bias rows from the per-row-tile column sums that the Gram kernel leaves behind:
//     u[i, q] = sum_tt upart[i, tt, q]  (tt ascending),   s_i (+)= sum_q u[i, q]^2.
// One workgroup of 1024 threads per example; thread t takes columns t, t + 1024, ... (the loads of a column's
// tiles are independent, four in flight); the squares are added per thread in column order, then over each wave
// and over the 16 waves in a fixed order.
constexpr int kFoldThreads = 1024;
__global__ __launch_bounds__(kFoldThreads) void k_bias_fold(const float* __restrict__ upart, int nt, int D, int accumulate,
                                                            float* __restrict__ u, float* __restrict__ sqnorm) {
    __shared__ float red[kFoldThreads / kWave];
    const int ex = blockIdx.x, tid = threadIdx.x;
    const float* p = upart + (size_t)ex * nt * D;
    float acc = 0.f;
    for (int q = tid; q < D; q += kFoldThreads) {
        float v = 0.f;
        int tt = 0;
        for (; tt + 3 < nt; tt += 4) {
            const float v0 = p[(size_t)tt * D + q], v1 = p[(size_t)(tt + 1) * D + q];
            const float v2 = p[(size_t)(tt + 2) * D + q], v3 = p[(size_t)(tt + 3) * D + q];
            v += v0; v += v1; v += v2; v += v3;
        }
        for (; tt < nt; ++tt) v += p[(size_t)tt * D + q];
        u[(size_t)ex * D + q] = v;
        acc += v * v;
    }
    acc = wave_sum(acc);
    if ((tid & (kWave - 1)) == 0) red[tid >> 6] = acc;
    __syncthreads();
    if (tid == 0) {
        float t = 0.f;
#pragma unroll
        for (int w = 0; w < kFoldThreads / kWave; ++w) t += red[w];
        sqnorm[ex] = accumulate ? sqnorm[ex] + t : t;
    }
}

hipError_t launch_bias_fold(const float* upart, int B, int nt, int D, bool accumulate, float* u, float* sqnorm, hipStream_t st) {
    k_bias_fold<<<(unsigned)B, kFoldThreads, 0, st>>>(upart, nt, D, accumulate ? 1 : 0, u, sqnorm);
    return hipGetLastError();
}

hipError_t launch_rows_sqnorm(const float* u, int B, int D, bool accumulate, float* sqnorm, hipStream_t st, const float* u2) {
    const int per_block = kThreads / kWave;
    k_rows_sqnorm<<<(unsigned)((B + per_block - 1) / per_block), kThreads, 0, st>>>(u, u2, B, D, accumulate ? 1 : 0, sqnorm);
    return hipGetLastError();
}

hipError_t launch_clipped_bias(const float* u, const float* clip, int B, int D, bool accumulate, float* grad_b, hipStream_t st) {
    if (B >= 2048) k_clipped_bias<32><<<(unsigned)((D + 31) / 32), 1024, 0, st>>>(u, clip, B, D, accumulate ? 1 : 0, grad_b);
    else           k_clipped_bias<8><<<(unsigned)((D + 31) / 32), kThreads, 0, st>>>(u, clip, B, D, accumulate ? 1 : 0, grad_b);
    return hipGetLastError();
}

hipError_t launch_bias_sqnorm_layers(const BiasLayerDesc* layers, int n_layers, int B, int dt, bool accumulate, float* sqnorm, hipStream_t st) {
    if (n_layers < 1 || n_layers > kBiasLayers || B < 1 || B > 65535 || dt < 0 || dt > 2) return hipErrorInvalidValue;
    BiasRowsLayers a;
    RowsLayers r;
    int64_t blocks = 0;
    const int vec = dt == 0 ? 4 : 8;
    for (int l = 0; l < kBiasLayers; ++l) {
        const BiasLayerDesc& y = layers[l < n_layers ? l : 0];
        const bool wide = y.D % vec == 0;
        a.G[l] = y.G; a.u[l] = y.u; a.T[l] = y.T; a.D[l] = y.D;
        a.ctl[l] = wide ? column_threads_log2(y.D / vec, B) : -1;
        a.chunks[l] = wide ? (y.D / vec + (1 << a.ctl[l]) - 1) >> a.ctl[l] : ceil_div(y.D, kScalarColumns);
        a.first_block[l] = (int)blocks;
        if (l < n_layers) blocks += (int64_t)a.chunks[l] * B;
        if (blocks >= (int64_t(1) << 24)) return hipErrorInvalidValue;
        r.u[l] = y.u; r.D[l] = y.D;
    }
    a.n_layers = r.n_layers = n_layers;
    if (dt == 0)      k_bias_rows_layers<0><<<(unsigned)blocks, kThreads, 0, st>>>(a);
    else if (dt == 1) k_bias_rows_layers<1><<<(unsigned)blocks, kThreads, 0, st>>>(a);
    else              k_bias_rows_layers<2><<<(unsigned)blocks, kThreads, 0, st>>>(a);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    k_rows_sqnorm_layers<<<(unsigned)B, kThreads, 0, st>>>(r, accumulate ? 1 : 0, sqnorm);
    return hipGetLastError();
}

hipError_t launch_clipped_bias_layers(const ClippedBiasDesc* layers, int n_layers, int B, bool accumulate, float stddev, uint64_t seed, hipStream_t st) {
    if (n_layers < 1 || n_layers > kBiasLayers || B < 1) return hipErrorInvalidValue;
    ClippedBiasLayers a;
    int64_t blocks = 0;
    for (int l = 0; l < kBiasLayers; ++l) {
        const ClippedBiasDesc& y = layers[l < n_layers ? l : 0];
        a.u[l] = y.u; a.clip[l] = y.clip; a.grad_b[l] = y.grad_b; a.noise_offset[l] = y.noise_offset; a.D[l] = y.D;
        a.first_block[l] = (int)blocks;
        if (l < n_layers) blocks += ceil_div(y.D, 32);       // widths are below 2^24: fewer than 2^23 workgroups
    }
    a.n_layers = n_layers;
    const NoiseArgs nz{stddev, (uint32_t)seed, (uint32_t)(seed >> 32), 0};
    if (B >= 2048) {
        if (blocks >= (int64_t(1) << 22)) return hipErrorInvalidValue;
        k_clipped_bias_layers<32><<<(unsigned)blocks, 1024, 0, st>>>(a, B, accumulate ? 1 : 0, nz);
    } else {
        k_clipped_bias_layers<8><<<(unsigned)blocks, kThreads, 0, st>>>(a, B, accumulate ? 1 : 0, nz);
    }
    return hipGetLastError();
}

}  // namespace dpk
