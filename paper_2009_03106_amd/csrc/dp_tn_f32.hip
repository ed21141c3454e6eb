// float32 K-major products  P = sum_k A[k, m-tile]^T G[k, n-tile]  on the
// fp32 MFMA (v_mfma_f32_32x32x2_f32).  That instruction takes one k per lane
// (lanes 0-31: k, lanes 32-63: k+1), so the K-major tiles are used as they lie
// in memory: LDS holds [k][col] and consecutive lanes read consecutive floats.
// Same two uses as the bf16 file: clipped sum (rows of A scaled by their
// example's clip factor, exactly, in fp32) and direct squared norm.
#include <algorithm>
#include <vector>
#include "dp_common.h"
#include "dp_internal.h"

namespace dpk {

namespace {

// k rows per stage: 64 where the contraction is long enough (a stage costs a global-load latency and two barriers
// whatever its size, so short stages make the loop latency-bound), 16 for short ones (direct norm of short sequences,
// where a 64-row stage would be mostly zero padding)
inline int stage_rows(int64_t k) { return k >= 128 ? 64 : 16; }
constexpr int FBM = 64, FBN = 64;     // block tile; 2 x 2 waves, one 32 x 32 MFMA tile each

struct TnArgsF {
    const float* A;
    const float* G;
    const float* clip;
    float* out;
    int64_t slice;
    int K, T, M, N;
    int tiles_m, tiles_n;
    int kchunk;
    int accumulate;
    int slices_per_example = 1;     // mode 2
};

// The loads of a stage are issued unconditionally from clamped (valid) addresses and zeroed afterwards: no branch
// sits between them, so they are all in flight together (a guarded load costs one memory round trip each).
// VECA / VECG: d_in / d_out is a multiple of 4, so every 16-byte piece of that operand is all inside or all outside a
// row and is one load; otherwise a piece is four 4-byte loads (each operand by itself: a 256 -> 10 classifier head
// still reads its wide operand in 16-byte pieces).
template <int MODE, int FBK, bool VECA, bool VECG>
__global__ __launch_bounds__(kThreads) void k_tn_f32(TnArgsF a) {
    constexpr int NV = FBK / 16;        // float4 pieces of either operand per thread and stage
    __shared__ __attribute__((aligned(16))) float sA[FBK][FBM];
    __shared__ __attribute__((aligned(16))) float sG[FBK][FBN];
    __shared__ float red[4];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int tile = blockIdx.x;
    const int tm = tile / a.tiles_n, tn = tile % a.tiles_n;
    const int m0 = tm * FBM, n0 = tn * FBN;
    const int z = blockIdx.y;
    int k_begin, k_end;
    if (MODE == 0) { k_begin = z * a.kchunk; k_end = min(a.K, k_begin + a.kchunk); }
    else if (MODE == 2) {
        // slice z = (example, chunk of its positions), its share of A_i^T G_i stored unscaled (direct norm of few long
        // examples of a small layer, see plan_direct_chunks)
        const int ex = z / a.slices_per_example, ch = z - ex * a.slices_per_example;
        k_begin = ex * a.T + ch * a.kchunk;
        k_end = min(ex * a.T + a.T, k_begin + a.kchunk);
    }
    else { k_begin = z * a.T; k_end = k_begin + a.T; }

    // each thread moves NV float4 of A and of G per stage: rows lr, lr + 16, ..., columns lc .. lc + 3 of the tile
    const int lr = tid >> 4;            // 0..15
    const int lc = (tid & 15) * 4;
    bool okA[4], okG[4];                // the column lies inside the matrix
    int colA[4], colG[4];               // a valid column to load from
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        okA[j] = m0 + lc + j < a.M; okG[j] = n0 + lc + j < a.N;
        colA[j] = okA[j] ? m0 + lc + j : 0; colG[j] = okG[j] ? n0 + lc + j : 0;
    }

    const int wm = wave >> 1, wn = wave & 1;
    const int lrow = lane & 31, lhalf = lane >> 5;
    f32x16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;

    float xa[NV][4], xg[NV][4];         // what fetch() loaded; scaled and zeroed in commit(), one stage of MFMAs
    float cl[NV];                       // later, so that the loads stay in flight behind them
    bool inr[NV];                       // the row lies inside the slice
    auto fetch = [&](int k0) {
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            const int row = k0 + lr + 16 * v;
            inr[v] = row < k_end;
            const int rc = inr[v] ? row : k_end - 1;                    // k_begin < k_end whenever a stage is fetched
            const float* pa = a.A + (size_t)rc * a.M;
            const float* pg = a.G + (size_t)rc * a.N;
            if (VECA) {
                const float4 qa = *reinterpret_cast<const float4*>(pa + colA[0]);
                xa[v][0] = qa.x; xa[v][1] = qa.y; xa[v][2] = qa.z; xa[v][3] = qa.w;
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j) xa[v][j] = pa[colA[j]];
            }
            if (VECG) {
                const float4 qg = *reinterpret_cast<const float4*>(pg + colG[0]);
                xg[v][0] = qg.x; xg[v][1] = qg.y; xg[v][2] = qg.z; xg[v][3] = qg.w;
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j) xg[v][j] = pg[colG[j]];
            }
            cl[v] = (MODE == 0) ? a.clip[a.T == 1 ? rc : rc / a.T] : 1.0f;
        }
    };
    auto commit = [&]() {
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            float ya[4], yg[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                ya[j] = (inr[v] && okA[j]) ? xa[v][j] * cl[v] : 0.f;
                yg[j] = (inr[v] && okG[j]) ? xg[v][j] : 0.f;
            }
            *reinterpret_cast<float4*>(&sA[lr + 16 * v][lc]) = make_float4(ya[0], ya[1], ya[2], ya[3]);
            *reinterpret_cast<float4*>(&sG[lr + 16 * v][lc]) = make_float4(yg[0], yg[1], yg[2], yg[3]);
        }
    };

    if (k_begin < k_end) fetch(k_begin);
    for (int k0 = k_begin; k0 < k_end; k0 += FBK) {
        commit();
        __syncthreads();
        if (k0 + FBK < k_end) fetch(k0 + FBK);
        // the operands of 8 MFMAs are read together, so that their LDS latency is paid once per group
#pragma unroll
        for (int k8 = 0; k8 < FBK / 2; k8 += 8) {
            float fa[8], fb[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                fa[j] = sA[(k8 + j) * 2 + lhalf][wm * 32 + lrow];
                fb[j] = sG[(k8 + j) * 2 + lhalf][wn * 32 + lrow];
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int j = 0; j < 8; ++j) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[j], fb[j], acc, 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
        __syncthreads();
    }

    if (MODE == 0 || MODE == 2) {
        float* out = a.out + (size_t)z * a.slice;
        const int n = n0 + wn * 32 + lrow;
        if (n < a.N) {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int m = m0 + wm * 32 + 8 * (r >> 2) + 4 * lhalf + (r & 3);
                if (m < a.M) {
                    float* p = out + (size_t)m * a.N + n;
                    *p = a.accumulate ? *p + acc[r] : acc[r];
                }
            }
        }
    } else {
        float s = 0.f;                  // columns outside the matrix are left out: an infinity times their zeros is NaN there
        const bool inn = n0 + wn * 32 + lrow < a.N;
#pragma unroll
        for (int r = 0; r < 16; ++r)
            s += inn && m0 + wm * 32 + 8 * (r >> 2) + 4 * lhalf + (r & 3) < a.M ? acc[r] * acc[r] : 0.f;
        s = block_sum_256(s, red);
        if (tid == 0) a.out[(size_t)z * (a.tiles_m * a.tiles_n) + tile] = s;
    }
}

// Clipped sum over a short contraction (dense layers: K = B, a few hundred rows): 32 x 32 output tile per workgroup,
// the four waves split the rows of every 64-row stage between them (wave w: rows 16 w .. 16 w + 15) and their four
// partial tiles are added through LDS in the order w = 0 .. 3.  The fp32 MFMA is a chain of dependent 64-cycle
// instructions per wave, so the 64 x 64 kernel above, one wave per 32 x 32 tile, needs K / 2 of them in a row and
// fills only (d_in / 64)(d_out / 64) compute units; here a wave runs K / 8 and there are four times as many
// workgroups.  No K slices: the whole sum is finished in the kernel.
constexpr int SBK = 64, STM = 32, STN = 32;
#define SHORT_LDS                                                          \
    __shared__ __attribute__((aligned(16))) float sA[SBK][STM];            \
    __shared__ __attribute__((aligned(16))) float sG[SBK][STN];            \
    __shared__ __attribute__((aligned(16))) float part[4][STM][STN + 1]
template <bool VECA, bool VECG>
__device__ __forceinline__ void tn_f32_short_tile(const TnArgsF& a, int tile, float (*sA)[STM], float (*sG)[STN],
                                                  float (*part)[STM][STN + 1]) {
    constexpr int NV = 2;               // float4 pieces of either operand per thread and stage

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int tm = tile / a.tiles_n, tn = tile % a.tiles_n;
    const int m0 = tm * STM, n0 = tn * STN;
    const int k_end = a.K;

    // each thread moves NV float4 of A and of G per stage: rows lr, lr + 32, columns lc .. lc + 3 of the tile
    const int lr = tid >> 3;            // 0..31
    const int lc = (tid & 7) * 4;
    bool okA[4], okG[4];
    int colA[4], colG[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        okA[j] = m0 + lc + j < a.M; okG[j] = n0 + lc + j < a.N;
        colA[j] = okA[j] ? m0 + lc + j : 0; colG[j] = okG[j] ? n0 + lc + j : 0;
    }
    const int lrow = lane & 31, lhalf = lane >> 5;
    f32x16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;

    // The loads of GS stages (256 rows: a whole contraction of the dense configurations) are issued before any of
    // them is used, so that a workgroup waits for memory once per 256 rows and not once per stage: with K = B = 256
    // the kernel is one memory latency, four short MFMA chains and the epilogue.
    constexpr int GS = 4;
    float xa[GS][NV][4], xg[GS][NV][4], cl[GS][NV];
    auto fetch = [&](int g, int k0) {
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            const int row = k0 + lr + 32 * v;
            const int rc = row < k_end ? row : k_end - 1;
            const float* pa = a.A + (size_t)rc * a.M;
            const float* pg = a.G + (size_t)rc * a.N;
            if (VECA) {
                const float4 qa = *reinterpret_cast<const float4*>(pa + colA[0]);
                xa[g][v][0] = qa.x; xa[g][v][1] = qa.y; xa[g][v][2] = qa.z; xa[g][v][3] = qa.w;
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j) xa[g][v][j] = pa[colA[j]];
            }
            if (VECG) {
                const float4 qg = *reinterpret_cast<const float4*>(pg + colG[0]);
                xg[g][v][0] = qg.x; xg[g][v][1] = qg.y; xg[g][v][2] = qg.z; xg[g][v][3] = qg.w;
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j) xg[g][v][j] = pg[colG[j]];
            }
            cl[g][v] = a.clip[a.T == 1 ? rc : rc / a.T];
        }
    };
    auto commit = [&](int g, int k0) {
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            const bool inr = k0 + lr + 32 * v < k_end;
            float ya[4], yg[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                ya[j] = (inr && okA[j]) ? xa[g][v][j] * cl[g][v] : 0.f;
                yg[j] = (inr && okG[j]) ? xg[g][v][j] : 0.f;
            }
            *reinterpret_cast<float4*>(&sA[lr + 32 * v][lc]) = make_float4(ya[0], ya[1], ya[2], ya[3]);
            *reinterpret_cast<float4*>(&sG[lr + 32 * v][lc]) = make_float4(yg[0], yg[1], yg[2], yg[3]);
        }
    };

    for (int kg = 0; kg < k_end; kg += GS * SBK) {
#pragma unroll
        for (int g = 0; g < GS; ++g)
            if (kg + g * SBK < k_end) fetch(g, kg + g * SBK);
#pragma unroll
        for (int g = 0; g < GS; ++g) {
            const int k0 = kg + g * SBK;
            if (k0 >= k_end) break;
            commit(g, k0);
            __syncthreads();
            float fa[8], fb[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                fa[j] = sA[wave * 16 + j * 2 + lhalf][lrow];
                fb[j] = sG[wave * 16 + j * 2 + lhalf][lrow];
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int j = 0; j < 8; ++j) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[j], fb[j], acc, 0, 0, 0);
            __syncthreads();
        }
    }

    // accumulator element r of a lane: row 8 (r / 4) + 4 lhalf + r % 4, column lrow of the 32 x 32 tile
#pragma unroll
    for (int r = 0; r < 16; ++r) part[wave][8 * (r >> 2) + 4 * lhalf + (r & 3)][lrow] = acc[r];
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int idx = tid + 256 * e;              // 1024 outputs, 4 per thread; consecutive threads: consecutive columns
        const int mr = idx >> 5, nc = idx & 31;
        const int m = m0 + mr, n = n0 + nc;
        if (m < a.M && n < a.N) {
            const float v = ((part[0][mr][nc] + part[1][mr][nc]) + part[2][mr][nc]) + part[3][mr][nc];
            float* p = a.out + (size_t)m * a.N + n;
            *p = a.accumulate ? *p + v : v;
        }
    }
}

// 16-byte loads for each operand whose width allows them (a 256 -> 10 head must not cost a wide layer its loads,
// nor its own wide operand)
__device__ __forceinline__ void tn_f32_short_dispatch(const TnArgsF& a, int tile, float (*sA)[STM], float (*sG)[STN],
                                                      float (*part)[STM][STN + 1]) {
    const bool va = (a.M & 3) == 0, vg = (a.N & 3) == 0;
    if (va) { if (vg) tn_f32_short_tile<true, true>(a, tile, sA, sG, part); else tn_f32_short_tile<true, false>(a, tile, sA, sG, part); }
    else    { if (vg) tn_f32_short_tile<false, true>(a, tile, sA, sG, part); else tn_f32_short_tile<false, false>(a, tile, sA, sG, part); }
}
__global__ __launch_bounds__(kThreads) void k_tn_f32_short(TnArgsF a) {
    SHORT_LDS;
    tn_f32_short_dispatch(a, blockIdx.x, sA, sG, part);
}

// The same for several layers in one launch (a model of small dense layers is a chain of launches of a few
// microseconds each otherwise): the layers' tiles form one list, in the order given.
constexpr int kShortBatch = 8;
struct TnShortLayers { int n_layers; int first_tile[kShortBatch + 1]; TnArgsF layer[kShortBatch]; };
__global__ __launch_bounds__(kThreads) void k_tn_f32_short_layers(TnShortLayers t) {
    SHORT_LDS;
    int li = 0;
    while (li + 1 < t.n_layers && (int)blockIdx.x >= t.first_tile[li + 1]) ++li;
    const TnArgsF a = t.layer[li];
    tn_f32_short_dispatch(a, (int)blockIdx.x - t.first_tile[li], sA, sG, part);
}

// Clipped sum of many rows with one narrow operand, at most 32 columns: a classifier head, the 27 patch columns of a first
// convolution.  It is bound by reading the wide operand, so nothing goes through LDS on the way: 32 consecutive columns of
// two rows are an operand of the 32 x 32 x 2 instruction as a wave's 4-byte loads bring them, the narrow one is loaded and
// scaled once for WT blocks of the wide one, and a wave has the loads of 2 U rows in flight.  A workgroup of 8 waves takes
// WT x 32 wide columns and a slice of the rows, a wave an eighth of it; their sums meet in LDS, three steps.  (64 x 64 tiles
// were mostly padding, 8 stages one after the other: 65536 rows of 256 x 10 took 36 us, the fold among them, now 24; with
// 256 columns a workgroup 31, their sums take longer to meet, with 32 rows in flight a wave 25.)
// SWAP: the narrow operand is A.  DT: 0 = float32, 1 = bf16, 2 = fp16; 16-bit inputs are widened as they come, so their products
// with the factors are exact to float32 too.
constexpr int kSkinnyThreads = 512;
constexpr int kSkinnyPairs = 8;                     // U
template <int DT> struct SkinnyElem { typedef uint16_t type; };
template <> struct SkinnyElem<0> { typedef float type; };
template <int WT, bool SWAP, int DT>
__global__ __launch_bounds__(kSkinnyThreads, 2) void k_tn_f32_skinny(TnArgsF a) {
    typedef typename SkinnyElem<DT>::type Elem;
    auto widen = [](Elem x) -> float {
        if constexpr (DT == 0) return x;
        else return In16<DT == 2>::lo((uint32_t)x);
    };
    constexpr int U = kSkinnyPairs;
    __shared__ float part[4][WT * 32][33];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 31, half = lane >> 5;
    const Elem* wide = reinterpret_cast<const Elem*>(SWAP ? a.G : a.A);
    const Elem* narrow = reinterpret_cast<const Elem*>(SWAP ? a.A : a.G);
    const int dw = SWAP ? a.N : a.M, dn = SWAP ? a.M : a.N;
    const int w0 = blockIdx.x * WT * 32, z = blockIdx.y;
    const int per_wave = a.kchunk / 8;
    const int k_begin = (int)min((int64_t)a.K, (int64_t)z * a.kchunk + (int64_t)wave * per_wave), k_end = (int)min((int64_t)a.K, (int64_t)k_begin + per_wave);
    int cw[WT];                                          // columns outside the matrices feed sums that are never stored
#pragma unroll
    for (int t = 0; t < WT; ++t) cw[t] = min(w0 + t * 32 + col, dw - 1);
    const int cn = min(col, dn - 1);
    f32x16 acc[WT];
#pragma unroll
    for (int t = 0; t < WT; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[t][r] = 0.f;
    for (int k0 = k_begin; k0 < k_end; k0 += 2 * U) {
        const bool full = k0 + 2 * U <= k_end;           // uniform
        const Elem* pw = wide + (size_t)k0 * dw;
        const Elem* pn = narrow + (size_t)k0 * dn;
        Elem w[U][WT], n[U];
        float c[U];
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const int r = min(2 * j + half, k_end - 1 - k0);          // rows past the end read the last one
#pragma unroll
            for (int t = 0; t < WT; ++t) w[j][t] = pw[(uint32_t)(r * dw + cw[t])];
            n[j] = pn[(uint32_t)(r * dn + cn)];
            c[j] = a.T == 1 ? a.clip[k0 + r] : 0.f;
        }
        if (a.T != 1) {
            const int ex = k0 / a.T;                     // uniform; one factor where the rows are of one example
            const float one = a.clip[ex];
            if ((min(k0 + 2 * U, k_end) - 1) / a.T == ex) {
#pragma unroll
                for (int j = 0; j < U; ++j) c[j] = one;
            } else {
#pragma unroll
                for (int j = 0; j < U; ++j) c[j] = a.clip[(k0 + min(2 * j + half, k_end - 1 - k0)) / a.T];
            }
        }
        if (!full) {                                     // ... and give zeros (both: an infinity times zero is NaN)
#pragma unroll
            for (int j = 0; j < U; ++j) {
                const bool in = k0 + 2 * j + half < k_end;
#pragma unroll
                for (int t = 0; t < WT; ++t) w[j][t] = in ? w[j][t] : (Elem)0;
                n[j] = in ? n[j] : (Elem)0;
                c[j] = in ? c[j] : 0.f;
            }
        }
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const float x = widen(n[j]) * c[j];
#pragma unroll
            for (int t = 0; t < WT; ++t) acc[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(widen(w[j][t]), x, acc[t], 0, 0, 0);
        }
    }
    auto put = [&](float (*to)[33]) {
#pragma unroll
        for (int t = 0; t < WT; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r) to[t * 32 + 8 * (r >> 2) + 4 * half + (r & 3)][col] = acc[t][r];
    };
    auto add = [&](float (*from)[33]) {
#pragma unroll
        for (int t = 0; t < WT; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[t][r] += from[t * 32 + 8 * (r >> 2) + 4 * half + (r & 3)][col];
    };
#pragma unroll
    for (int n = 4; n >= 1; n >>= 1) {
        if (wave >= n && wave < 2 * n) put(part[wave - n]);
        __syncthreads();
        if (wave < n) add(part[wave]);
        __syncthreads();
    }
    if (wave == 0) put(part[0]);
    __syncthreads();
    const int rows = min(WT * 32, dw - w0);
    float* out = a.out + (size_t)z * a.slice;
    for (int e = tid; e < rows * dn; e += kSkinnyThreads) {
        const int i = SWAP ? e % rows : e / dn, k = SWAP ? e / rows : e - i * dn;       // wide and narrow column
        float* p = out + (SWAP ? (size_t)k * dw + w0 + i : (size_t)(w0 + i) * dn + k);
        const float v = part[0][i][k];
        *p = a.accumulate ? *p + v : v;
    }
}

// blocks of 32 wide columns per workgroup
inline int skinny_blocks(int dw) {
    const int groups = ceil_div(dw, 128);
    return ceil_div(ceil_div(dw, 32), groups) <= 2 ? 2 : 4;
}
template <bool SWAP, int DT> void launch_skinny_dt(int blocks, dim3 grid, const TnArgsF& a, hipStream_t st) {
    if (blocks == 2) k_tn_f32_skinny<2, SWAP, DT><<<grid, kSkinnyThreads, 0, st>>>(a);
    else             k_tn_f32_skinny<4, SWAP, DT><<<grid, kSkinnyThreads, 0, st>>>(a);
}
template <bool SWAP> void launch_skinny(int blocks, dim3 grid, const TnArgsF& a, int dt, hipStream_t st) {
    if (dt == 0)      launch_skinny_dt<SWAP, 0>(blocks, grid, a, st);
    else if (dt == 1) launch_skinny_dt<SWAP, 1>(blocks, grid, a, st);
    else              launch_skinny_dt<SWAP, 2>(blocks, grid, a, st);
}

template <int MODE, int FBK> void launch_f32_k(bool veca, bool vecg, dim3 grid, const TnArgsF& a, hipStream_t st) {
    if (veca) { if (vecg) k_tn_f32<MODE, FBK, true, true><<<grid, kThreads, 0, st>>>(a); else k_tn_f32<MODE, FBK, true, false><<<grid, kThreads, 0, st>>>(a); }
    else      { if (vecg) k_tn_f32<MODE, FBK, false, true><<<grid, kThreads, 0, st>>>(a); else k_tn_f32<MODE, FBK, false, false><<<grid, kThreads, 0, st>>>(a); }
}
template <int MODE> void launch_f32(bool deep, bool veca, bool vecg, dim3 grid, const TnArgsF& a, hipStream_t st) {
    if (deep) launch_f32_k<MODE, 64>(veca, vecg, grid, a, st);
    else      launch_f32_k<MODE, 16>(veca, vecg, grid, a, st);
}

}  // namespace

// The geometry on which a layer's sum can run on the split kernel.  Up to kShortK rows only outputs of at least 64 tiles
// of 128 x 128, which fill the chip without K slices.
int clipped_f32_split_geo(int64_t K, int M, int N) {
    if (K >= (int64_t(1) << 31)) return F32_NONE;
    if (K <= kShortK && (int64_t)ceil_div(M, 128) * ceil_div(N, 128) < 64) return F32_NONE;
    return f32_split_geo(K, M, N, false);
}

// Where the split kernel is the faster one for a layer by itself, in products K M N (us, fp32 kernels / split):
//   up to kShortK rows from 1e9:  844 x 1664 from 384 20 / 29, 768 x 2304 from 512 28 / 34; 4608 x 512 from 512 37 / 36,
//                                 2000 x 2000 from 256 35 / 33
//   sizes that are no multiple of 4 (the fp32 kernel loads their rows word by word) from 1.5e8:  63 x 127 from 6000
//                                 22 / 24, from 25000 53 / 43
//   aligned shapes of 128 x 128 tiles always: 128 x 128 from 520 29 / 15 (the kernel it replaced)
//   one aligned tile of 64 columns never: 64 x 128 from 25000 14 / 18, from 100000 31 / 32, from 400000 88 / 94
//   others from 3.7e8:            576 x 64 from 6000 14 / 19, 64 x 256 from 12500 14 / 17, 250 x 60 from 25000 24 / 22
ClippedF32Route clipped_f32_route(int64_t K, int M, int N) {
    const int geo = clipped_f32_split_geo(K, M, N);
    const double products = (double)K * M * N;
    if (K <= kShortK) return geo != F32_NONE && products >= 1e9 ? ClippedF32Route{false, geo} : ClippedF32Route{true, F32_NONE};
    if (geo == F32_NONE) return ClippedF32Route{false, F32_NONE};
    const bool aligned = ((M | N) & 3) == 0;
    const int64_t pm = (int64_t)ceil_div(M, 128) * 128, pn = (int64_t)ceil_div(N, 128) * 128;
    bool split;
    if (aligned && pm * pn * 3 <= (int64_t)M * N * 4) split = true;
    else if ((((int64_t)M * N) & 3) != 0) split = products >= 1.5e8;
    else if (aligned && M <= f32_split_tile_m(geo) && N <= f32_split_tile_n(geo)) split = false;
    else split = products >= 3.7e8;
    return ClippedF32Route{false, split ? geo : F32_NONE};
}

// A sum that the kernel of one narrow operand takes (of those that are neither short nor the split kernel's).  The line, in
// us (64 x 64 tiles / this kernel): one group of columns 64 x 10 from 4096 rows 12.5 / 12.7, 27 x 64 from 32768 13.9 / 11.3;
// rows of odd length, which the tiles load word by word, 139 x 2 from 4096 16.9 / 13.0; else by the wide operand's entries:
// 256 x 10 from 16384 rows 13.5 / 13.9, from 65536 36.2 / 24.4; 512 x 20 from 8192 12.2 / 14.2, from 10963 17.6 / 15.7;
// 1024 x 10 from 4096 13.2 / 13.6, from 10963 26.9 / 20.4; 784 x 32 from 10963 21.9 / 21.1, from 65536 93 / 61.
bool plan_skinny(TnPlan& p, int64_t K, int M, int N) {
    const int dw = std::max(M, N);
    if (std::min(M, N) > 32 || dw > (1 << 20) || K < 4096 || K >= (int64_t(1) << 31) - 4096) return false;
    if (dw > 128 && (dw & 3) == 0 && K * dw < 4500000) return false;
    // one workgroup per compute unit: slices of at least 2 U rows a wave
    const int blocks = skinny_blocks(dw), least = 8 * 2 * kSkinnyPairs;
    p.skinny = true;
    p.segmented = false; p.epu = 0; p.big = false; p.dma = false; p.zero_head = false;
    p.tile_m = M >= N ? blocks * 32 : 32; p.tile_n = M >= N ? 32 : blocks * 32;
    p.tiles_m = ceil_div(M, p.tile_m); p.tiles_n = ceil_div(N, p.tile_n);
    const int64_t groups = (int64_t)p.tiles_m * p.tiles_n;
    const int64_t want = groups >= 256 ? 1 : 256 / groups;
    const int64_t kchunk = ceil_div(ceil_div(K, want), least) * (int64_t)least;
    p.kchunk = (int)kchunk;
    p.splits = (int)((K + kchunk - 1) / kchunk);
    return true;
}

hipError_t launch_clipped_skinny(const TnPlan& p, const void* A, const void* G, const float* clip, int B, int T, int M, int N, bool accumulate,
                                 float* grad, float* ws, hipStream_t st, int dt, const NoiseArgs* noise) {
    TnArgsF a;
    a.A = static_cast<const float*>(A); a.G = static_cast<const float*>(G); a.clip = clip;
    a.K = B * T; a.T = T; a.M = M; a.N = N;
    a.tiles_m = p.tiles_m; a.tiles_n = p.tiles_n; a.kchunk = p.kchunk;
    const int64_t n = (int64_t)M * N;
    if (p.splits == 1) { a.out = grad; a.slice = 0; a.accumulate = accumulate ? 1 : 0; }
    else { a.out = ws; a.slice = splitk_slice_elems(n); a.accumulate = 0; }
    dim3 grid((unsigned)(p.tiles_m * p.tiles_n), (unsigned)p.splits);
    if (M < N) launch_skinny<true>(p.tile_n / 32, grid, a, dt, st);
    else       launch_skinny<false>(p.tile_m / 32, grid, a, dt, st);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || p.splits == 1) return e;
    return launch_splitk_reduce(ws, n, p.splits, accumulate, grad, st, noise);
}

TnPlan plan_clipped_f32(int B, int T, int M, int N) {
    const int64_t K = (int64_t)B * T;
    TnPlan p;
    p.segmented = false; p.epu = 0; p.big = false; p.dma = false;
    const ClippedF32Route route = clipped_f32_route(K, M, N);
    const int geo = route.geo;
    if (route.is_short) {
        p.tile_m = STM; p.tile_n = STN;
        p.tiles_m = ceil_div(M, STM); p.tiles_n = ceil_div(N, STN);
        p.splits = 1; p.kchunk = (int)K;
        return p;
    }
    if (geo != F32_NONE) {
        // 4-wave geometries: two workgroups per compute unit, 256 x 256: one; slices of at least 4 stages
        const int dk = f32_split_stage_rows();
        const int slots_log2 = geo == F32_BIG ? 8 : 9;
        p.dma = true;
        p.tile_m = f32_split_tile_m(geo); p.tile_n = f32_split_tile_n(geo);
        p.tiles_m = ceil_div(M, p.tile_m); p.tiles_n = ceil_div(N, p.tile_n);
        const int64_t tiles = (int64_t)p.tiles_m * p.tiles_n;
        // K slices: the (tile, slice) items run `slots` at a time; an item costs its stages plus about 16 stage times of
        // start-up and store, and the fold reads all slices, 4 MB in about a stage time, and walks them one after the
        // other, 32 (k_splitk_reduce_wide) or 4 (k_splitk_reduce) in a stage time.  (Sizes that are no multiple of 4 are counted
        // at 4, though the wide fold takes them too: with 32 they would take up to twice the slices and scratch for 0.9 % of the
        // time, 60 sizes between 0.92 and 1.5.)  Take the slice count with the
        // smallest rounds x (stages per slice + 16) + fold: a count that just spills into one more round (540 items)
        // costs a whole extra round, many short slices cost their overheads.
        const uint32_t stages = (uint32_t)((K + dk - 1) / dk);
        uint32_t max_splits = stages / 4;
        if (max_splits < 1) max_splits = 1;
        if (max_splits > 256) max_splits = 256;
        const uint32_t walked = splitk_reduce_is_wide((int64_t)M * N) ? 32 : 4;
        uint32_t best = 1;
        int64_t best_cost = -1;
        for (uint32_t sp = 1; sp <= max_splits;) {
            const uint32_t sps = (stages + sp - 1) / sp, real = (stages + sps - 1) / sps;
            const int64_t rounds = (tiles * real + (1 << slots_log2) - 1) >> slots_log2;
            const int64_t cost = rounds * (sps + 16) + ((real * (int64_t)M * N) >> 20) + real / walked;
            if (best_cost < 0 || cost < best_cost) { best_cost = cost; best = sp; }
            if (sps == 1) break;
            sp = (stages + sps - 2) / (sps - 1);             // the next count whose slices are shorter
        }
        const int64_t kchunk = (int64_t)((stages + best - 1) / best) * dk;
        p.kchunk = (int)kchunk;
        p.splits = (int)((K + kchunk - 1) / kchunk);
        return p;
    }
    if (plan_skinny(p, K, M, N)) return p;
    p.tile_m = FBM; p.tile_n = FBN;
    p.tiles_m = ceil_div(M, FBM); p.tiles_n = ceil_div(N, FBN);
    const int64_t tiles = (int64_t)p.tiles_m * p.tiles_n;
    const int FBK = stage_rows(K);
    int64_t want = (512 + tiles - 1) / tiles;
    int64_t max_splits = (K + 4 * FBK - 1) / (4 * FBK);      // at least 4 stages per slice
    if (want > max_splits) want = max_splits;
    if (want < 1) want = 1;
    int64_t kchunk = (K + want - 1) / want;
    kchunk = ((kchunk + FBK - 1) / FBK) * FBK;
    if (kchunk < FBK) kchunk = FBK;
    p.kchunk = (int)kchunk;
    p.splits = (int)((K + kchunk - 1) / kchunk);
    if (p.splits < 1) p.splits = 1;
    return p;
}

// Which kernel forms a direct norm.  The split kernel (dp_tn_f32_split.hip) walks an example in one workgroup per tile; the
// fp32 kernel above has smaller tiles, a shorter way from stage to stage, and cuts the positions of few long examples
// into chunks: B = 1 .. 16, T = 12544, 64 x 128 takes 29 .. 57 us there and 510 us on the split kernel, B = 512 takes 1.2 ms
// and 0.95 ms.  The two are compared by their times in us, fitted to measurements of 13 shapes of 60 .. 1152 columns,
// T = 128 .. 12544, B = 1 .. 512 (880 points: what is chosen takes 0.3 % longer than the faster one in the mean):
//   split   a row of the longest example takes 0.041 us, 0.045 us where the launch has an item for every compute unit, and
//           more in proportion from two per compute unit on; an item of 128 x 128 counts as one and a half
//   fp32    rounds of 256 items, 0.022 us a row and 1.7 us an item, rows of unaligned widths up to 1.6 times as long;
//           in chunks 18 us and the products' time
// Aligned shapes of 128 x 128 tiles go to the split kernel from T = 256 on.
namespace {
bool direct_f32_always_split(int T, int M, int N) {
    const int64_t pm = (int64_t)ceil_div(M, 128) * 128, pn = (int64_t)ceil_div(N, 128) * 128;
    return T >= 256 && ((M | N) & 3) == 0 && pm * pn * 3 <= (int64_t)M * N * 4;
}
// rows that a layer's items walk
double direct_f32_split_rows(int B, int T, int M, int N) {
    const int geo = f32_split_geo(T, M, N, true);
    const double items = (double)B * ceil_div(M, f32_split_tile_m(geo)) * ceil_div(N, f32_split_tile_n(geo));
    return items * T * (geo == F32_MID ? 1.5 : 1.0);
}
double direct_f32_split_us(double longest, double rows) {
    const double items = rows / longest;
    const double row = items <= 256 ? 0.041 + 0.004 * items / 256 : items <= 512 ? 0.045 + 0.028 * (items - 256) / 256 : 0.073 * items / 512;
    return 6.2 + longest * row;
}
TnPlan plan_direct_f32_fp32(int B, int T, int M, int N) {
    TnPlan p;
    p.segmented = false; p.epu = 0; p.big = false; p.dma = false;
    p.tile_m = FBM; p.tile_n = FBN;
    p.tiles_m = ceil_div(M, FBM); p.tiles_n = ceil_div(N, FBN);
    p.splits = 1; p.kchunk = 0;
    plan_direct_chunks(p, B, T, M, N, 4, 64);
    return p;
}
double direct_f32_fp32_us(int B, int T, int M, int N) {
    const TnPlan p = plan_direct_f32_fp32(B, T, M, N);
    const int odd = ((M & 3) != 0) + ((N & 3) != 0);
    if (p.splits > 1) return 18.0 + (double)B * T * M * N / (odd == 0 ? 4.2e7 : odd == 1 ? 3.1e7 : 2.5e7);
    const double row = odd == 0 ? 0.0222 : odd == 1 ? 0.030 : 0.0365;
    return 5.5 + ceil_div((int64_t)B * p.tiles_m * p.tiles_n, 256) * (1.7 + row * T);
}
}  // namespace

// Several layers in one launch (every layer has a geometry of the split kernel): take[l] = 0 for the layers that are left
// to launches of their own.  Those are the longest ones, as many as makes the whole fastest: the launch takes as long
// as its longest example, and saves the others a launch each.
void choose_direct_f32_joint(const JointShape* sh, int n_layers, int B, char* take) {
    std::vector<int> order;
    double rows = 0.0, fixed = 0.0;                          // fixed: the longest of the layers that stay in any case
    for (int l = 0; l < n_layers; ++l) {
        take[l] = 1;
        rows += direct_f32_split_rows(B, sh[l].T, sh[l].M, sh[l].N);
        if (direct_f32_always_split(sh[l].T, sh[l].M, sh[l].N)) fixed = std::max(fixed, (double)sh[l].T);
        else order.push_back(l);
    }
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return sh[a].T > sh[b].T; });
    size_t best = 0;
    double best_us = -1.0, alone = 0.0;
    for (size_t k = 0; k <= order.size(); ++k) {             // the k longest on their own
        const double longest = std::max(fixed, k < order.size() ? (double)sh[order[k]].T : 0.0);
        const double us = alone + (longest > 0.0 ? direct_f32_split_us(longest, rows) : 0.0);
        if (best_us < 0.0 || us < best_us) { best_us = us; best = k; }
        if (k == order.size()) break;
        const JointShape& s = sh[order[k]];
        alone += direct_f32_fp32_us(B, s.T, s.M, s.N);
        rows -= direct_f32_split_rows(B, s.T, s.M, s.N);
    }
    for (size_t k = 0; k < best; ++k) take[order[k]] = 0;
}

TnPlan plan_direct_f32(int B, int T, int M, int N) {
    const int geo = f32_split_geo(T, M, N, true);
    if (geo != F32_NONE && (direct_f32_always_split(T, M, N) ||
                            direct_f32_split_us(T, direct_f32_split_rows(B, T, M, N)) <= direct_f32_fp32_us(B, T, M, N))) {
        TnPlan p;
        p.segmented = false; p.epu = 0; p.big = false; p.dma = true;
        p.tile_m = f32_split_tile_m(geo); p.tile_n = f32_split_tile_n(geo);
        p.tiles_m = ceil_div(M, p.tile_m); p.tiles_n = ceil_div(N, p.tile_n);
        p.splits = 1; p.kchunk = 0;
        return p;
    }
    return plan_direct_f32_fp32(B, T, M, N);
}

hipError_t launch_clipped_f32(const TnPlan& p, const float* A, const float* G, const float* clip,
                              int B, int T, int M, int N, bool accumulate, float* grad, float* ws, hipStream_t st,
                              const NoiseArgs* noise) {
    TnArgsF a;
    a.A = A; a.G = G; a.clip = clip;
    a.K = B * T; a.T = T; a.M = M; a.N = N;
    a.tiles_m = p.tiles_m; a.tiles_n = p.tiles_n; a.kchunk = p.kchunk;
    const int64_t n = (int64_t)M * N;
    if (p.splits == 1) { a.out = grad; a.slice = 0; a.accumulate = accumulate ? 1 : 0; }
    else { a.out = ws; a.slice = splitk_slice_elems(n); a.accumulate = 0; }
    if (p.dma) {
        hipError_t e = launch_tn_f32_split(0, p, A, G, clip, B, T, M, N, a.out, a.slice, a.accumulate != 0, st);
        if (e != hipSuccess || p.splits == 1) return e;
        return launch_splitk_reduce(ws, n, p.splits, accumulate, grad, st, noise);
    }
    if (p.skinny) return launch_clipped_skinny(p, A, G, clip, B, T, M, N, accumulate, grad, ws, st, 0, noise);
    if (p.tile_m == STM) {
        a.out = grad; a.slice = 0; a.accumulate = accumulate ? 1 : 0;
        const unsigned tiles = (unsigned)(p.tiles_m * p.tiles_n);
        k_tn_f32_short<<<tiles, kThreads, 0, st>>>(a);
        return hipGetLastError();
    }
    dim3 grid((unsigned)(p.tiles_m * p.tiles_n), (unsigned)p.splits);
    launch_f32<0>(stage_rows(a.K) == 64, (M & 3) == 0, (N & 3) == 0, grid, a, st);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || p.splits == 1) return e;
    return launch_splitk_reduce(ws, n, p.splits, accumulate, grad, st, noise);
}


hipError_t launch_clipped_f32_short_layers(const ShortLayerDesc* layers, int n_layers, int B, bool accumulate, hipStream_t st) {
    if (n_layers < 1 || n_layers > kShortBatch) return hipErrorInvalidValue;
    TnShortLayers t;
    t.n_layers = n_layers;
    int64_t first = 0;
    // the layers that cannot use 16-byte loads first: their workgroups take about twice as long, and the workgroups of
    // a launch start in the order of their ids (536 of them for the MLP configuration start over several microseconds)
    int order[kShortBatch], no = 0;
    for (int pass = 0; pass < 2; ++pass)
        for (int l = 0; l < n_layers; ++l)
            if ((((layers[l].M | layers[l].N) & 3) != 0) == (pass == 0)) order[no++] = l;
    for (int l = 0; l < kShortBatch; ++l) {
        t.first_tile[l] = (int)first;
        if (l >= n_layers) { t.layer[l] = TnArgsF{nullptr, nullptr, nullptr, nullptr, 0, 0, 1, 0, 0, 0, 0, 0, 0}; continue; }
        const ShortLayerDesc& y = layers[order[l]];
        TnArgsF& a = t.layer[l];
        a.A = y.A; a.G = y.G; a.clip = y.clip;
        a.K = B * y.T; a.T = y.T; a.M = y.M; a.N = y.N;
        a.tiles_m = ceil_div(y.M, STM); a.tiles_n = ceil_div(y.N, STN); a.kchunk = a.K;
        a.out = y.grad; a.slice = 0; a.accumulate = accumulate ? 1 : 0;
        first += (int64_t)a.tiles_m * a.tiles_n;
        if (first >= (int64_t(1) << 31)) return hipErrorInvalidValue;
    }
    t.first_tile[kShortBatch] = (int)first;
    k_tn_f32_short_layers<<<(unsigned)first, kThreads, 0, st>>>(t);
    return hipGetLastError();
}

hipError_t launch_direct_f32(const TnPlan& p, const float* A, const float* G, int B, int T, int M, int N,
                             bool accumulate, float* sqnorm, float* partial, hipStream_t st, const ClipOut* co) {
    TnArgsF a;
    a.clip = nullptr;
    a.K = B * T; a.T = T; a.M = M; a.N = N;
    a.tiles_m = p.tiles_m; a.tiles_n = p.tiles_n; a.kchunk = 0;
    a.slice = 0; a.accumulate = 0;
    const int tiles = p.tiles_m * p.tiles_n;
    if (p.dma) {
        // one launch of (example, tile) items; batches of more than a launch holds go in pieces
        const int64_t per = std::max<int64_t>(1, (int64_t(1) << 22) / tiles);
        for (int64_t b0 = 0; b0 < B; b0 += per) {
            const int nb = (int)((B - b0 < per) ? (B - b0) : per);
            hipError_t e = launch_tn_f32_split(1, p, A + (size_t)b0 * T * M, G + (size_t)b0 * T * N, nullptr, nb, T, M, N,
                                             partial + (size_t)b0 * tiles, 0, false, st);
            if (e != hipSuccess) return e;
        }
        return launch_finalize_partials(partial, B, tiles, accumulate, sqnorm, st, co);
    }
    if (p.splits > 1) {
        // chunks of positions: workspace = the chunks' shares [B][S][slice], then sums[B][nblk]
        const int64_t n = (int64_t)M * N, slice = splitk_slice_elems(n);
        const int nblk = (int)((n + 1023) / 1024);
        float* sums = partial + (size_t)B * p.splits * slice;
        a.A = A; a.G = G;
        a.kchunk = p.kchunk; a.out = partial; a.slice = slice; a.slices_per_example = p.splits;
        dim3 grid((unsigned)tiles, (unsigned)(B * p.splits));
        launch_f32<2>(true, (M & 3) == 0, (N & 3) == 0, grid, a, st);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        e = launch_direct_chunks_finish(partial, slice, p.splits, (int)n, B, sums, st);
        if (e != hipSuccess) return e;
        return launch_finalize_partials(sums, B, nblk, accumulate, sqnorm, st, co);
    }
    for (int b0 = 0; b0 < B; b0 += 65535) {
        const int nb = (B - b0 < 65535) ? (B - b0) : 65535;
        a.A = A + (size_t)b0 * T * M;
        a.G = G + (size_t)b0 * T * N;
        a.out = partial + (size_t)b0 * tiles;
        dim3 grid((unsigned)tiles, (unsigned)nb);
        launch_f32<1>(stage_rows(T) == 64, (M & 3) == 0, (N & 3) == 0, grid, a, st);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return launch_finalize_partials(partial, B, tiles, accumulate, sqnorm, st, co);
}

}  // namespace dpk
