// float32 K-major products  P = sum_k A[k, m-tile]^T G[k, n-tile]  for long contractions, on the bf16 MFMA with every
// operand split into three bf16 numbers (dp_split.h): the rate of the fp32 MFMA (157 TFLOP/s nominal) bounded these
// sums, six bf16 products have 2.7 times that.
//   * The workgroup splits each element once, on its way into LDS: a thread loads the 8 rows of K of one column
//     (4-byte loads, 64 consecutive columns per wave; 4 rows of the operand of 64 columns), so that the packed halves are
//     the MFMA operand as it stands, 16 bytes that go to LDS with one write per part and are read back with one read
//     per fragment, both without bank conflicts.  4-byte loads also take any width and alignment.
//   * 16-row stages, two in LDS; the loads of the stage after next wait in registers, one barrier per stage.
//   * The clip factors of a stage's rows are the same for a whole wave: scalar loads, multiplied into the A values
//     before the split (the same a * c rounded once to float32 as in the row-scaling kernels; the split's scale is in
//     the factor).  Rows past the end of the K slice come back from the buffer loads as zeros.
// Two uses, as in the 16-bit file: clipped sum (Eq. weighted_loss) over K slices, and direct squared norm (Algorithm
// 3 / 4 without their output tensor): the slice is one example and the finished tile is squared and summed.
#include <algorithm>
#include "dp_common.h"
#include "dp_internal.h"
#include "dp_split.h"

namespace dpk {

namespace {

constexpr int DKF = 16;                 // rows of K per stage: one MFMA deep

// Geometry: WM x WN waves, each with MI x NI tiles of 32 x 32.
template <int MI_, int NI_, int WM_, int WN_> struct GeoF {
    static constexpr int MI = MI_, NI = NI_, WM = WM_, WN = WN_;
    static constexpr int TM = WM * MI * 32, TN = WN * NI * 32, THREADS = 64 * WM * WN;
    static constexpr int STAGE_UNITS = 2 * 3 * (TM + TN);      // 16-byte units: [part][k / 8][column], A then G
    // one column of A and of G per thread, 2 PA and 2 PG rows of it: two or four threads take a column
    static constexpr int PA = 8 * TM / THREADS, PG = 8 * TN / THREADS;
    static_assert((PA == 4 || PA == 2) && (PG == 4 || PG == 2) && TM % 64 == 0 && TN % 64 == 0, "");
};
using GeoBig = GeoF<4, 2, 2, 4>;        // 256 x 256, 8 waves
using GeoMid = GeoF<2, 2, 2, 2>;        // 128 x 128, 4 waves, as the next two: layers of these three share a launch
using GeoNarrow = GeoF<2, 1, 2, 2>;     // 128 x 64: a convolution of 64 channels
using GeoFlat = GeoF<1, 2, 2, 2>;       // 64 x 128

struct F32SplitArgs {
    const float* A;
    const float* G;
    const float* clip;
    float* out;            // slice base (stride `slice` per K slice) or grad; direct norm: partial[B][tiles]
    int64_t slice;
    int K, T, M, N;
    int tiles_m, tiles_n;
    int splits;            // K slices (direct norm: examples)
    int kchunk;            // rows per K slice, a multiple of DKF
    int per_xcd;
    int accumulate;
};

// The wave's sums once more with the float32 instruction, in the order of k: for sums of 2^80 and more, infinities and
// NaN (see dp_split.h).  Straight from memory and slow.
template <int MODE, int MI, int NI>
__device__ __forceinline__ void tn_f32_exact(const F32SplitArgs& a, int k_begin, int k_end, int mw, int nw, f32x16 (&acc)[MI][NI]) {
    const int lrow = threadIdx.x & 31, lhalf = (threadIdx.x & 63) >> 5;
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    for (int k = k_begin; k < k_end; k += 2) {
        const bool in = k + lhalf < k_end;                   // an odd last row: the other half of the lanes gives zeros
        const int row = in ? k + lhalf : k_end - 1;
        const float c = MODE == 0 ? a.clip[row / a.T] : 1.0f;
        float fa[MI], fg[NI];
#pragma unroll
        for (int i = 0; i < MI; ++i) {
            const float x = a.A[(size_t)row * a.M + min(mw + i * 32 + lrow, a.M - 1)] * c;
            fa[i] = in ? x : 0.f;
        }
#pragma unroll
        for (int j = 0; j < NI; ++j) {
            const float x = a.G[(size_t)row * a.N + min(nw + j * 32 + lrow, a.N - 1)];
            fg[j] = in ? x : 0.f;
        }
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NI; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[i], fg[j], acc[i][j], 0, 0, 0);
    }
}

// MODE 0: clipped sum over K slice z = rows [z kchunk, (z + 1) kchunk).  MODE 1: direct squared norm of example z.
// The rows of a wave.  256 x 256 tiles: the blocks of 32 rows are dealt evenly to the tiles, a tile's to its two rows of waves:
// 784 rows are 25 blocks in tiles of 6 and 7, where four whole tiles would form 32 (65536 rows of 784 x 512: 31 % of the
// products for nothing).  (f32_split_geo takes these tiles where at most a quarter is padding, so every tile has 6 to 8.)
struct WaveRows { int m0, first, blocks; };            // first row of the tile, of the wave inside it, the wave's blocks
template <class GEO> __device__ __forceinline__ WaveRows wave_rows(const F32SplitArgs& a, int tm, int wm) {
    if constexpr (GEO::MI == 4) {
        const int blocks = (a.M + 31) / 32;
        const int b0 = (int)((int64_t)tm * blocks / a.tiles_m), b1 = (int)((int64_t)(tm + 1) * blocks / a.tiles_m);
        const int upper = (b1 - b0 + 1) / 2;
        return {b0 * 32, wm == 0 ? 0 : upper * 32, wm == 0 ? upper : b1 - b0 - upper};
    } else {
        return {tm * GEO::TM, wm * GEO::MI * 32, GEO::MI};
    }
}
// tile of item L's (slice, tile)
__device__ __forceinline__ void tile_of(const F32SplitArgs& a, int tile, int& tm, int& tn) {
    if (a.tiles_m < a.tiles_n) { tn = tile / a.tiles_m; tm = tile - tn * a.tiles_m; }       // the short side of the tile grid first
    else { tm = tile / a.tiles_n; tn = tile - tm * a.tiles_n; }
}

// One wave's part of item L of the launch, (slice, tile), slice-major: MI blocks of 32 rows
template <int MODE, class GEO, int MI>
__device__ __forceinline__ void tn_f32_split_wave(const F32SplitArgs& a, const int L, u32x4* lds) {
    constexpr int NI = GEO::NI, TM = GEO::TM, TN = GEO::TN, SU = GEO::STAGE_UNITS, PA = GEO::PA, PG = GEO::PG;

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tiles = a.tiles_m * a.tiles_n;
    if (L >= (int64_t)tiles * a.splits) return;
    const int z = L / tiles, tile = L - z * tiles;
    int tm, tn;
    tile_of(a, tile, tm, tn);
    const WaveRows rows = wave_rows<GEO>(a, tm, wave / GEO::WN);
    const int m0 = rows.m0, n0 = tn * TN, mofs = rows.first;
    int k_begin, k_end;
    if (MODE == 0) { k_begin = z * a.kchunk; k_end = min(a.K, k_begin + a.kchunk); }
    else { k_begin = z * a.T; k_end = k_begin + a.T; }
    const int n_stages = (k_end - k_begin + DKF - 1) / DKF;
    if (n_stages <= 0) return;

    // ---- global -> registers -> LDS: a thread moves rows r0 .. r0 + 2 P - 1 of the stage, one column of either operand.
    //      r0A and r0G are the same for a whole wave.  Columns outside the matrix only feed outputs that are never stored.
    const int r0A = __builtin_amdgcn_readfirstlane(tid / TM) * (2 * PA), r0G = __builtin_amdgcn_readfirstlane(tid / TN) * (2 * PG);
    const uint32_t wrA = (uint32_t)((r0A >> 3) * TM + tid % TM), wrG = (uint32_t)(6 * TM + (r0G >> 3) * TN + tid % TN);   // units of part 0
    // buffer loads: a row past the end of the slice lies outside the buffer and comes back as zero
    const uint32_t rowA = (uint32_t)a.M * 4u, rowG = (uint32_t)a.N * 4u;
    const uint32_t offA = (uint32_t)min(m0 + tid % TM, a.M - 1) * 4u, offG = (uint32_t)min(n0 + tid % TN, a.N - 1) * 4u;
    float ra[2 * PA], rg[2 * PG], rc = 1.0f;
    // lane l: the factor of row l % (2 PA) of the wave's rows of the stage
    int fex = 0, fpos = 0;                               // example and position inside it of that row, next stage
    const int last_ex = MODE == 0 ? (k_end - 1) / a.T : 0;
    if (MODE == 0) { const int row = k_begin + r0A + (lane & (2 * PA - 1)); fex = row / a.T; fpos = row - fex * a.T; }
    const int adv_ex = DKF / a.T, adv_pos = DKF - adv_ex * a.T;
    int next_a = k_begin + r0A, next_g = k_begin + r0G;
    // The MFMA rounds its sums down, which in long sums of random sign adds up (K = 65536: 5.6e-7 of the result): every other
    // stage is formed with the sign of A turned and subtracted, so that the two errors cancel.
    float sign_a = 1.0f;                                 // of the next stage to fetch
    uint32_t at_a = 0, at_g = 0;
    auto fetch = [&](bool of_a, int q) {                 // rows 2 q and 2 q + 1 of one operand of the next stage, in order of q
        const int next_row = of_a ? next_a : next_g;
        const int nrows = __builtin_amdgcn_readfirstlane(max(0, min(of_a ? 2 * PA : 2 * PG, k_end - next_row)));
        if (of_a) {
            if (q == 0) at_a = offA;
            asm volatile("" : "+v"(at_a));               // 16 offsets kept from stage to stage would not fit the registers
            const auto buf = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.A + (size_t)next_row * a.M), (short)0, (int)(nrows * rowA), 0x00020000);
            ra[2 * q] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(buf, at_a, 0, 0)); at_a += rowA;
            ra[2 * q + 1] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(buf, at_a, 0, 0)); at_a += rowA;
            if (q < PA - 1) return;
            if (MODE == 0) {
                rc = a.clip[min(fex, last_ex)] * (sign_a * kSplitScale);
                sign_a = -sign_a;
                fex += adv_ex; fpos += adv_pos;
                if (fpos >= a.T) { fpos -= a.T; ++fex; }
            }
            next_a += DKF;
            return;
        }
        if (q == 0) at_g = offG;
        asm volatile("" : "+v"(at_g));
        const auto buf = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(a.G + (size_t)next_row * a.N), (short)0, (int)(nrows * rowG), 0x00020000);
        rg[2 * q] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(buf, at_g, 0, 0)); at_g += rowG;
        rg[2 * q + 1] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(buf, at_g, 0, 0)); at_g += rowG;
        if (q == PG - 1) next_g += DKF;
    };
    // the split in PA + PG steps, rows 2 q and 2 q + 1 of A, then of G; each requests its rows of the stage after, the last of
    // either writes the operand's parts to LDS
    u32x4 parts[3];
    auto split_step = [&](int pair, int buf) {
        const bool of_a = pair < PA;
        const int q = of_a ? pair : pair - PA;
        float x0, x1;
        if (of_a) {
            x0 = ra[2 * q]; x1 = ra[2 * q + 1];
            if (MODE == 0) {
                x0 *= __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(rc), 2 * q));
                x1 *= __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(rc), 2 * q + 1));
            } else { x0 *= kSplitScale; x1 *= kSplitScale; }
        } else { x0 = rg[2 * q] * kSplitScale; x1 = rg[2 * q + 1] * kSplitScale; }
        uint32_t p1, p2, p3;
        split2(x0, x1, p1, p2, p3);
        parts[0][q] = p1; parts[1][q] = p2; parts[2][q] = p3;
        if (q == (of_a ? PA : PG) - 1) {
#pragma unroll
            for (int p = 0; p < 3; ++p) {
                u32x4* to = lds + (buf * SU + (of_a ? p * 2 * TM + wrA : p * 2 * TN + wrG));
                if ((of_a ? PA : PG) == 4) *to = parts[p];
                else reinterpret_cast<uint2*>(to)[((of_a ? r0A : r0G) >> 2) & 1] = make_uint2(parts[p][0], parts[p][1]);
            }
        }
        fetch(of_a, q);                                  // in the place of the two that were split
    };

    // ---- LDS -> MFMA operands: lane (lrow, lhalf) takes column lrow of a 32-wide block and rows 8 lhalf .. 8 lhalf + 7
    const int wn = wave % GEO::WN;
    const int lrow = lane & 31, lhalf = lane >> 5;
    const uint32_t rdA = (uint32_t)(lhalf * TM + mofs + lrow);
    const uint32_t rdG = (uint32_t)(6 * TM + lhalf * TN + wn * NI * 32 + lrow);

    f32x16 acc[MI][NI];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

#pragma unroll
    for (int q = 0; q < PA; ++q) fetch(true, q);
#pragma unroll
    for (int q = 0; q < PG; ++q) fetch(false, q);
#pragma unroll
    for (int q = 0; q < PA + PG; ++q) split_step(q, 0);
    __builtin_amdgcn_s_waitcnt(0xC07F);
    __builtin_amdgcn_s_barrier();
    // Past the end of the slice the copies bring zeros, which nobody reads: the loop has no branches.  One 32 x 32 tile
    // of the wave after the other: its six MFMAs, in their shadow a share of the next stage's split and the addition
    // of the tile before.  (With the split in front of all MFMAs the two add up: the waves of a workgroup are in step.)
    constexpr int TILES = MI * NI;                       // the PA + PG steps of the split are dealt to them in turn
    constexpr int STEPS = (PA + PG) / TILES;
    f32x16 pend = {};                                    // the sums of the tile before, not yet added
    // The 4-wave geometries keep their sums in two levels, blocks of 8 stages and their sum (four layers 576 -> 64, 32768
    // rows: 1.16e-7 of the result off, 1.85e-7 without; 128 x 128 then takes 250 registers and not 180, two workgroups
    // per compute unit in both cases).
    constexpr bool TWO = MODE == 0 && GEO::MI * GEO::NI <= 4;
    f32x16 total[TWO ? MI : 1][TWO ? NI : 1];
    if constexpr (TWO) {
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NI; ++j) total[i][j] = f32x16{};
    }
    for (int st = 0; st < n_stages; ++st) {
        const int buf = st & 1;
        const float sign = MODE == 0 && buf ? -kSplitUnscale : kSplitUnscale;
        bf16x8 fg[NI][3], fa[2][3];
        auto read_a = [&](int i) {
#pragma unroll
            for (int p = 0; p < 3; ++p) fa[i & 1][p] = __builtin_bit_cast(bf16x8, lds[buf * SU + rdA + p * 2 * TM + i * 32]);
        };
        read_a(0);
#pragma unroll
        for (int j = 0; j < NI; ++j)
#pragma unroll
            for (int p = 0; p < 3; ++p) fg[j][p] = __builtin_bit_cast(bf16x8, lds[buf * SU + rdG + p * 2 * TN + j * 32]);
#pragma unroll
        for (int t = 0; t < TILES; ++t) {
            const int i = t / NI, j = t % NI, before = (t + TILES - 1) % TILES;
            if (j == 0 && i + 1 < MI) read_a(i + 1);
            acc[before / NI][before % NI] += pend * (MODE == 0 && t == 0 ? -sign : sign);
            pend = split_mfma(fa[i & 1], fg[j]);
#pragma unroll
            for (int q = 0; q < (PA + PG + TILES - 1) / TILES; ++q) {
                const int k = t * (PA + PG) / TILES + q;
                if (k < (t + 1) * (PA + PG) / TILES) split_step(k, buf ^ 1);
            }
#pragma unroll
            for (int q = 0; q < 6; ++q) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x002, STEPS == 1 ? 5 : STEPS == 2 ? 7 : 9, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        __builtin_amdgcn_s_waitcnt(0xC07F);              // lgkmcnt(0): this wave's parts of the next stage are in LDS
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (TWO) {
            if ((st & 7) == 7) {
#pragma unroll
                for (int i = 0; i < MI; ++i)
#pragma unroll
                    for (int j = 0; j < NI; ++j) { total[i][j] += acc[i][j]; acc[i][j] = f32x16{}; }
            }
        }
    }
    acc[MI - 1][NI - 1] += pend * (MODE == 0 && !(n_stages & 1) ? -kSplitUnscale : kSplitUnscale);
    if constexpr (TWO) {
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NI; ++j) acc[i][j] += total[i][j];
    }

    const int mw = m0 + mofs, nw = n0 + wn * NI * 32;
    SplitCheck check;
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) check.add(acc[i][j][r]);
    if (__any(check.suspect())) tn_f32_exact<MODE, MI, NI>(a, k_begin, k_end, mw, nw, acc);

    if (MODE == 1) {
        float sq = 0.f;
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NI; ++j) {
                const int n = nw + j * 32 + lrow;
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int m = mw + i * 32 + 8 * (r >> 2) + 4 * lhalf + (r & 3);
                    const float v = acc[i][j][r];
                    sq += (m < a.M && n < a.N) ? v * v : 0.f;
                }
            }
        sq = wave_sum(sq);
        float* red = reinterpret_cast<float*>(lds);      // every wave is past its last read of the stages (barrier above)
        if (lane == 0) red[wave] = sq;
        __syncthreads();
        if (tid == 0) {
            float s = 0.f;
#pragma unroll
            for (int w = 0; w < GEO::WM * GEO::WN; ++w) s += red[w];
            a.out[(size_t)z * tiles + tile] = s;
        }
        return;
    }
    float* out = a.out + (size_t)z * a.slice;
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) {
            const int n = nw + j * 32 + lrow;
            if (n >= a.N) continue;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int m = mw + i * 32 + 8 * (r >> 2) + 4 * lhalf + (r & 3);
                if (m < a.M) {
                    float* p = out + (size_t)m * a.N + n;
                    *p = a.accumulate ? *p + acc[i][j][r] : acc[i][j][r];
                }
            }
        }
}

template <int MODE, class GEO>
__device__ __forceinline__ void tn_f32_split_tile(const F32SplitArgs& a, const int L, u32x4* lds) {
    if constexpr (GEO::MI == 4) {
        const int tiles = a.tiles_m * a.tiles_n;
        int tm, tn;
        tile_of(a, L % tiles, tm, tn);
        if (wave_rows<GEO>(a, tm, __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6) / GEO::WN).blocks == 4)
            tn_f32_split_wave<MODE, GEO, 4>(a, L, lds);
        else
            tn_f32_split_wave<MODE, GEO, 3>(a, L, lds);
    } else {
        tn_f32_split_wave<MODE, GEO, GEO::MI>(a, L, lds);
    }
}

template <int MODE, class GEO>
__global__ __launch_bounds__(GEO::THREADS, 2) void k_tn_f32_split(F32SplitArgs a) {
    __shared__ u32x4 lds[2 * GEO::STAGE_UNITS];
    // workgroup b runs on XCD b % 8: each XCD takes a contiguous run of (slice, tile) items, slice-major, so that
    // its workgroups stream the same rows of A and G through one L2
    tn_f32_split_tile<MODE, GEO>(a, (blockIdx.x & 7) * a.per_xcd + (blockIdx.x >> 3), lds);
}

// Several layers' clipped sums in one launch, as for the 16-bit inputs (dp_tn_bf16_dma.hip): the launch is a list of
// (layer, K slice, tile) items, a layer's items slice-major, dealt to the XCDs in contiguous runs.
struct F32JointLayer {
    const float* A; const float* G; const float* clip;
    float* out;            // the layer's K slices; the gradient itself where one slice is the whole sum
    int K, T, M, N, tiles_m, tiles_n, splits, kchunk, first_item, accumulate, geo;
};
struct F32JointArgs {
    F32JointLayer layer[kJointLayers];
    int n_layers, n_items, per_xcd;
};
// MODE 1: the layers' direct squared norms (a layer's "K slices" are its examples, `out` is partial[B][tiles])
// BIG: all layers on 256 x 256 tiles; else each on one of the three geometries of 4 waves
template <int MODE, bool BIG>
__global__ __launch_bounds__(BIG ? GeoBig::THREADS : GeoMid::THREADS, 2) void k_tn_f32_split_joint(F32JointArgs j) {
    __shared__ u32x4 lds[2 * (BIG ? GeoBig::STAGE_UNITS : GeoMid::STAGE_UNITS)];
    // The layers' items differ in length, so every XCD takes its eighth of every layer's items (first_item: among the
    // items of one XCD): with eighths of the whole list 18 convolutions' sums took 1.2 times as long.  On 256 x 256 tiles
    // they have about one length: an eighth of the list.
    const int xcd = blockIdx.x & 7, L = BIG ? xcd * j.per_xcd + (int)(blockIdx.x >> 3) : (int)(blockIdx.x >> 3);
    if (L >= j.n_items) return;
    int l = 0;
    while (l + 1 < j.n_layers && L >= j.layer[l + 1].first_item) ++l;
    const F32JointLayer& y = j.layer[l];
    int item = L - y.first_item;
    if (!BIG) item += xcd * (((int64_t)y.tiles_m * y.tiles_n * y.splits + 7) / 8);
    F32SplitArgs a;
    a.A = y.A; a.G = y.G; a.clip = y.clip;
    a.out = y.out; a.slice = (((int64_t)y.M * y.N) + 3) & ~(int64_t)3;          // splitk_slice_elems
    a.K = y.K; a.T = y.T; a.M = y.M; a.N = y.N;
    a.tiles_m = y.tiles_m; a.tiles_n = y.tiles_n; a.splits = y.splits; a.kchunk = y.kchunk;
    a.per_xcd = 0; a.accumulate = y.accumulate;
    if constexpr (BIG)               tn_f32_split_tile<MODE, GeoBig>(a, item, lds);
    else if (y.geo == F32_MID)       tn_f32_split_tile<MODE, GeoMid>(a, item, lds);
    else if (y.geo == F32_NARROW)    tn_f32_split_tile<MODE, GeoNarrow>(a, item, lds);
    else                             tn_f32_split_tile<MODE, GeoFlat>(a, item, lds);
}

}  // namespace

// One slice length (in 16-row stages) for all layers of a joint launch, each layer rounding it to equal slices:
// minimise  rounds of 512 (256 x 256 tiles: 256) workgroups x (stages of the longest slice + what an item costs besides its stages) + the fold's
// reading of the slices (4 MB in about a stage time) and its walk through the layer with the most of them (8 in a stage time).
F32JointPlan plan_joint_f32(const JointShape* sh, int n_layers, int B, bool big, size_t max_floats) {
    constexpr int64_t kItemOverhead = 16;
    F32JointPlan p{};
    // layers with the same number of stages and slice length take the same number of slices: they are counted together
    struct { uint32_t stages; bool half; int64_t tiles, entries, slice; } same[kJointLayers];
    int n_same = 0, which[kJointLayers];
    uint32_t stages_max = 1;
    for (int l = 0; l < n_layers; ++l) {
        const int64_t K = (int64_t)B * sh[l].T, entries = (int64_t)sh[l].M * sh[l].N;
        p.geo[l] = big ? F32_BIG : clipped_f32_split_geo(K, sh[l].M, sh[l].N);
        p.tiles_m[l] = ceil_div(sh[l].M, f32_split_tile_m(p.geo[l])); p.tiles_n[l] = ceil_div(sh[l].N, f32_split_tile_n(p.geo[l]));
        const uint32_t stages = (uint32_t)ceil_div(K, DKF);
        const bool half = p.geo[l] == F32_NARROW || p.geo[l] == F32_FLAT;
        stages_max = std::max(stages_max, stages);
        int k = 0;
        while (k < n_same && (same[k].stages != stages || same[k].half != half)) ++k;
        if (k == n_same) { same[k].stages = stages; same[k].half = half; same[k].tiles = same[k].entries = same[k].slice = 0; ++n_same; }
        same[k].tiles += (int64_t)p.tiles_m[l] * p.tiles_n[l]; same[k].entries += entries; same[k].slice += splitk_slice_elems(entries);
        which[l] = k;
    }
    int64_t best_cost = -1;
    uint32_t splits[kJointLayers], sps[kJointLayers], best_splits[kJointLayers], best_sps[kJointLayers];
    for (uint32_t S = 1; S <= 512 && S <= stages_max;) {
        const uint32_t len = (stages_max + S - 1) / S;
        if (len < 4 && S > 1) break;
        int64_t items = 0, fold = 0;                         // fold: entries of all slices
        uint32_t longest = 0, most = 0;
        size_t floats = 0;
        for (int k = 0; k < n_same; ++k) {
            const uint32_t own = same[k].half ? len + len / 2 : len;          // half a tile: shorter stages
            const uint32_t want = (same[k].stages + own - 1) / own;
            sps[k] = (same[k].stages + want - 1) / want;
            splits[k] = (same[k].stages + sps[k] - 1) / sps[k];
            items += same[k].tiles * splits[k];
            fold += same[k].entries * splits[k];
            floats += (size_t)same[k].slice * splits[k];
            longest = std::max(longest, own == len ? sps[k] : sps[k] * 2 / 3);
            most = std::max(most, splits[k]);
        }
        if (floats > max_floats && S > 1) break;             // (as plan_joint)
        // in eighths of a stage; a launch of one workgroup per compute unit or less takes 7 / 8 of one with two
        const int64_t rounds = big ? ((items + 255) >> 8) * 8 : items <= 256 ? 7 : ((items + 511) >> 9) * 8;
        const int64_t cost = rounds * (longest + kItemOverhead) + (fold >> 17) + most;
        if (best_cost < 0 || cost < best_cost) {
            best_cost = cost; p.items = items; p.floats = floats;
            for (int k = 0; k < n_same; ++k) { best_splits[k] = splits[k]; best_sps[k] = sps[k]; }
        }
        if (len == 1) break;
        S = (stages_max + len - 2) / (len - 1);              // the next count whose slices are shorter
    }
    for (int l = 0; l < n_layers; ++l) { p.splits[l] = (int)best_splits[which[l]]; p.kchunk[l] = (int)best_sps[which[l]] * DKF; }
    return p;
}

// noise: stddev == 0 for none, else every layer's d_in * d_out and noise_offset are multiples of 4.  A, G of the
// operands are float pointers here.
hipError_t launch_clipped_f32_split_joint(const JointShape* sh, const JointOperands* op, int n_layers, int B, bool accumulate,
                                        float stddev, uint64_t seed, float* ws, hipStream_t st, bool big, const F32JointPlan& p) {
    if (n_layers < 1 || n_layers > kJointLayers) return hipErrorInvalidValue;
    if (p.items >= (int64_t(1) << 28)) return hipErrorInvalidValue;
    F32JointArgs j;
    FoldLayers f;
    int nf = 0;
    float* slices = ws;
    int64_t first = 0;
    for (int l = 0; l < n_layers; ++l) {
        F32JointLayer& y = j.layer[l];
        y.A = reinterpret_cast<const float*>(op[l].A); y.G = reinterpret_cast<const float*>(op[l].G); y.clip = op[l].clip;
        // one slice and no noise to add: the launch writes the gradient itself, nothing to fold
        const bool whole = p.splits[l] == 1 && stddev == 0.0f;
        y.out = whole ? op[l].grad : slices;
        y.accumulate = whole && accumulate ? 1 : 0;
        y.K = B * sh[l].T; y.T = sh[l].T; y.M = sh[l].M; y.N = sh[l].N;
        y.tiles_m = p.tiles_m[l]; y.tiles_n = p.tiles_n[l]; y.splits = p.splits[l]; y.kchunk = p.kchunk[l]; y.geo = p.geo[l];
        y.first_item = (int)first;
        first += big ? (int64_t)p.tiles_m[l] * p.tiles_n[l] * p.splits[l] : ceil_div((int64_t)p.tiles_m[l] * p.tiles_n[l] * p.splits[l], 8);
        if (!whole) {
            f.ws[nf] = slices; f.grad[nf] = op[l].grad; f.n[nf] = (int64_t)sh[l].M * sh[l].N;
            f.splits[nf] = p.splits[l]; f.noise_offset[nf] = op[l].noise_offset;
            ++nf;
        }
        slices += (size_t)p.splits[l] * (size_t)splitk_slice_elems((int64_t)sh[l].M * sh[l].N);
    }
    for (int l = n_layers; l < kJointLayers; ++l) j.layer[l] = j.layer[0];
    j.n_layers = n_layers; j.n_items = big ? (int)p.items : (int)first; j.per_xcd = big ? ceil_div(p.items, 8) : (int)first;
    if (big) k_tn_f32_split_joint<0, true><<<8u * (unsigned)j.per_xcd, GeoBig::THREADS, 0, st>>>(j);
    else     k_tn_f32_split_joint<0, false><<<8u * (unsigned)j.per_xcd, GeoMid::THREADS, 0, st>>>(j);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || nf == 0) return e;
    f.n_layers = nf;
    for (int l = nf; l < kJointLayers; ++l) { f.ws[l] = f.ws[0]; f.grad[l] = f.grad[0]; f.n[l] = 0; f.splits[l] = 0; f.noise_offset[l] = 0; }
    return launch_splitk_reduce_layers(f, accumulate, st, stddev, seed, true);
}

// The geometry of a layer: the largest tiles of which at most a quarter is padding.  256 x 256 tiles (clipped sums
// only: half the L2 traffic per product of 128 x 128 tiles and a third less LDS traffic) where they are many
// stages' work: B = 64, T = 512, 768 x 2304 / 768 / 3072 and 3072 x 768 take 2.36 .. 2.5 ms on them and 2.9 ms on 128 x
// 128 tiles, 65536 rows of 784 x 512 and 512 x 256 0.43 .. 0.51 and 0.50 .. 0.60 ms; small convolutions of 16 .. 1024
// positions are faster in one launch of the smaller tiles.  (Of the 256 registers that a lane of the 8 waves has, the
// sums take 128; 122 values are kept in scratch memory, 228 bytes a lane, some of them across the stage loop.)
int f32_split_geo(int64_t K, int M, int N, bool direct) {
    if (K < (direct ? 128 : 256)) return F32_NONE;
    auto fits = [&](int geo) {
        const int tm = f32_split_tile_m(geo), tn = f32_split_tile_n(geo);
        const int64_t pm = (int64_t)ceil_div(M, tm) * tm, pn = (int64_t)ceil_div(N, tn) * tn;
        return pm * pn * 3 <= (int64_t)M * N * 4;
    };
    if (!direct && fits(F32_BIG) && (int64_t)ceil_div(M, 256) * ceil_div(N, 256) * (K / DKF) >= 4096) return F32_BIG;
    if (fits(F32_MID)) return F32_MID;
    if (fits(F32_NARROW)) return F32_NARROW;
    if (fits(F32_FLAT)) return F32_FLAT;
    return F32_NONE;
}
int f32_split_tile_m(int geo) { return geo == F32_BIG ? GeoBig::TM : geo == F32_FLAT ? GeoFlat::TM : GeoMid::TM; }
int f32_split_tile_n(int geo) { return geo == F32_BIG ? GeoBig::TN : geo == F32_NARROW ? GeoNarrow::TN : GeoMid::TN; }
int f32_split_stage_rows() { return DKF; }

// mode 0: clipped sum, p.splits K slices of p.kchunk rows to out (+ z * slice); mode 1: direct norm, one item per
// (example, tile) to out[B][tiles].
hipError_t launch_tn_f32_split(int mode, const TnPlan& p, const float* A, const float* G, const float* clip, int B, int T,
                             int M, int N, float* out, int64_t slice, bool accumulate, hipStream_t st) {
    F32SplitArgs a;
    a.A = A; a.G = G; a.clip = clip; a.out = out; a.slice = slice;
    a.K = B * T; a.T = T; a.M = M; a.N = N;
    a.tiles_m = p.tiles_m; a.tiles_n = p.tiles_n;
    a.splits = mode == 0 ? p.splits : B;
    a.kchunk = mode == 0 ? p.kchunk : T;
    a.accumulate = accumulate ? 1 : 0;
    const int64_t items = (int64_t)p.tiles_m * p.tiles_n * a.splits;
    if (items <= 0 || !launch_holds((items + 7) / 8 * 8, p.tile_m == GeoBig::TM && mode == 0 ? GeoBig::THREADS : GeoMid::THREADS)) return hipErrorInvalidValue;
    if (mode == 0 && (p.kchunk % DKF) != 0) return hipErrorInvalidValue;
    a.per_xcd = (int)((items + 7) / 8);
    const unsigned grid = 8u * (unsigned)a.per_xcd;
    if (p.tile_m == GeoBig::TM && mode == 0) k_tn_f32_split<0, GeoBig><<<grid, GeoBig::THREADS, 0, st>>>(a);
    else if (p.tile_m == GeoFlat::TM) { if (mode == 0) k_tn_f32_split<0, GeoFlat><<<grid, GeoFlat::THREADS, 0, st>>>(a); else k_tn_f32_split<1, GeoFlat><<<grid, GeoFlat::THREADS, 0, st>>>(a); }
    else if (p.tile_n == GeoNarrow::TN) { if (mode == 0) k_tn_f32_split<0, GeoNarrow><<<grid, GeoNarrow::THREADS, 0, st>>>(a); else k_tn_f32_split<1, GeoNarrow><<<grid, GeoNarrow::THREADS, 0, st>>>(a); }
    else { if (mode == 0) k_tn_f32_split<0, GeoMid><<<grid, GeoMid::THREADS, 0, st>>>(a); else k_tn_f32_split<1, GeoMid><<<grid, GeoMid::THREADS, 0, st>>>(a); }
    return hipGetLastError();
}

// Several layers' direct norms in one launch; partial[l]: the layer's [B][tiles of f32_split_geo] sums of squares, to be
// added by the caller.  Every layer: f32_split_geo has a geometry for it.
hipError_t launch_direct_f32_split_joint(const JointShape* sh, const JointOperands* op, float* const* partial, int n_layers,
                                       int B, hipStream_t st) {
    if (n_layers < 1 || n_layers > kJointLayers) return hipErrorInvalidValue;
    F32JointArgs j;
    int64_t first = 0;
    for (int l = 0; l < n_layers; ++l) {
        F32JointLayer& y = j.layer[l];
        y.A = reinterpret_cast<const float*>(op[l].A); y.G = reinterpret_cast<const float*>(op[l].G); y.clip = nullptr;
        y.out = partial[l]; y.accumulate = 0;
        y.K = B * sh[l].T; y.T = sh[l].T; y.M = sh[l].M; y.N = sh[l].N;
        y.geo = f32_split_geo(sh[l].T, sh[l].M, sh[l].N, true);
        if (y.geo == F32_NONE) return hipErrorInvalidValue;
        y.tiles_m = ceil_div(sh[l].M, f32_split_tile_m(y.geo)); y.tiles_n = ceil_div(sh[l].N, f32_split_tile_n(y.geo));
        y.splits = B; y.kchunk = sh[l].T;
        y.first_item = (int)first;
        first += ceil_div((int64_t)y.tiles_m * y.tiles_n * B, 8);
    }
    if (!launch_holds(8 * first, GeoMid::THREADS)) return hipErrorInvalidValue;
    for (int l = n_layers; l < kJointLayers; ++l) j.layer[l] = j.layer[0];
    j.n_layers = n_layers; j.n_items = (int)first; j.per_xcd = 0;
    k_tn_f32_split_joint<1, false><<<8u * (unsigned)first, GeoMid::THREADS, 0, st>>>(j);
    return hipGetLastError();
}

}  // namespace dpk
