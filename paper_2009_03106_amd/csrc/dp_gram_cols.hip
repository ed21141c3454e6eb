// Gram path for the per-example squared norm of a layer whose weights are shared by T positions (Sections 5.2 and
// 5.3: g_i = A_i^T G_i; its squared Frobenius norm is the sum over position pairs of (A_i A_i^T)_{ts} (G_i G_i^T)_{ts})
// for layers of few positions (T <= 64) and wide rows in a small batch: the late
// convolutions of an image model (4 x 4 or 8 x 8 positions, 2304 -> 256 or 4608 -> 512 unfolded columns, 20 to 32
// examples).  One workgroup per example walks thousands of columns alone there and leaves most of the chip idle, so
// here the COLUMNS are split: every wave takes a range of the columns of A and G (one after the other), forms its
// share of A_i A_i^T and of G_i G_i^T, the four waves of a workgroup add their shares through LDS, and a second kernel
// adds the workgroups' shares of an example in a fixed order, multiplies the two T x T products entry by entry and sums.
//
// Both operands of a Gram product are rows of the same matrix, so a 16-byte piece of a row serves the left and the right
// side of the MFMA alike.  16-bit inputs: the piece (8 consecutive columns of one row) is one operand of the 32 x 32 x 16
// instruction (row = lane % 32, columns 8 * (lane / 32) .. + 7 of a 16-column step).  float32: the piece (4 columns) feeds
// four 32 x 32 x 2 instructions, entry j of lanes 0-31 and of lanes 32-63 being the two columns of the j-th; which columns
// meet in an instruction does not matter to the sum, and both sides use the same register.
//
// The pieces come through LDS: a copy instruction moves 8 rows x 128 bytes (global_load_lds_dwordx4), whole cache lines,
// into the wave's own 16 KB, from where a lane reads its row.  (Loaded straight to registers a lane needs the 16 bytes of
// its own row, an instruction touches 32 lines for 32 bytes each, and the launches moved 1.9 TB/s: 32 examples of 64
// positions into 2304 x 256, three layers, and 1152 x 256 took 19.4 us.  Eight layers of an 18-layer image model, 56 MB,
// take 15 us in one launch (3.8 TB/s) and 5 us for the sums; in two launches by registers, with a walk through the shares, 60 us.)
#include <algorithm>
#include "dp_common.h"
#include "dp_internal.h"

namespace dpk {

namespace {

constexpr int kColsSteps = 8;        // 32-byte steps of a row that a wave takes at least, in flight together
constexpr int kStageSteps = 4;       // steps of one copied stage: 128 bytes of every row
constexpr int kWaveLds = 16384;      // bytes of a wave's stages in a launch of several layers: 2 of 64 rows or 4 of 32 rows
constexpr int kStages1 = 4, kStages2 = 2;      // stages in flight at most, rows of one and of two 32-row blocks
#define LDS_PTR(T) __attribute__((address_space(3))) T*

struct GramColsLayer {
    const void* A;
    const void* G;
    float* sums;         // [B][tiles of the triangle]: the layer's sums (several layers only)
    size_t part_off;     // floats: where the layer's shares start in the scratch
    int T, d_in, d_out;
    int steps_a;         // steps (16 columns of 16-bit inputs, 8 of float32) of A; the steps of G follow them
    int steps;           // of A and G together
    int W;               // workgroups per example
    int per_wave;        // steps per wave
    int nb;              // 32-row blocks of positions: 1 (T <= 32) or 2
    unsigned first_block;
    unsigned first_finish;      // first workgroup of k_gram_cols_sums
};
// Several layers in one launch: a layer alone is a few hundred workgroups that each make one memory round trip, so the
// launches of a model's layers mostly wait.  CAP: the most layers (a layer alone does not pay for the arguments of 16).
template <int CAP> struct GramColsArgs {
    GramColsLayer layer[CAP];
    float* part;         // per layer [B][W][2][NT][4][64][4]: the workgroups' shares of the two products, in accumulator layout
    int n_layers;
    int wave_lds;        // bytes of a wave's stages
    int stages;          // of layers with one 32-row block: how many of them
};

// at most n of the wave's copies may still be in flight
__device__ __forceinline__ void wait_copies(int n) {
#define DP_WAIT(k) case k: asm volatile("s_waitcnt vmcnt(" #k ")" ::: "memory"); break;
    switch (n) {
        DP_WAIT(1) DP_WAIT(2) DP_WAIT(3) DP_WAIT(4) DP_WAIT(5) DP_WAIT(6) DP_WAIT(7) DP_WAIT(8) DP_WAIT(9) DP_WAIT(10) DP_WAIT(11) DP_WAIT(12)
        default: asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
#undef DP_WAIT
}

// acc[tile] += X[rows of block b0] . X[rows of block b1]^T for one step, a 16-byte piece per lane and block; tiles in the
// order (0,0), (0,1), (1,1) for two 32-row blocks.  FIRST: acc starts from zero.
template <int NB, int DT, bool FIRST = false>
__device__ __forceinline__ void gram_cols_mfma(const uint4 (&f)[NB], f32x16 (&acc)[NB * (NB + 1) / 2]) {
    constexpr f32x16 zero = {};
    if constexpr (DT == 0) {
        const float a0[4] = {__uint_as_float(f[0].x), __uint_as_float(f[0].y), __uint_as_float(f[0].z), __uint_as_float(f[0].w)};
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(a0[e], a0[e], FIRST && e == 0 ? zero : acc[0], 0, 0, 0);
        if constexpr (NB == 2) {
            const float a1[4] = {__uint_as_float(f[1].x), __uint_as_float(f[1].y), __uint_as_float(f[1].z), __uint_as_float(f[1].w)};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                acc[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(a0[e], a1[e], FIRST && e == 0 ? zero : acc[1], 0, 0, 0);
                acc[2] = __builtin_amdgcn_mfma_f32_32x32x2f32(a1[e], a1[e], FIRST && e == 0 ? zero : acc[2], 0, 0, 0);
            }
        }
    } else {
        constexpr bool F16 = DT == 2;
        const bf16x8 f0 = __builtin_bit_cast(bf16x8, f[0]);
        acc[0] = In16<F16>::mfma(f0, f0, FIRST ? zero : acc[0]);
        if constexpr (NB == 2) {
            const bf16x8 f1 = __builtin_bit_cast(bf16x8, f[1]);
            acc[1] = In16<F16>::mfma(f0, f1, FIRST ? zero : acc[1]);
            acc[2] = In16<F16>::mfma(f1, f1, FIRST ? zero : acc[2]);
        }
    }
}

// The steps [kb, ke) of X (an example's T rows of `row_bytes` bytes, a multiple of 16), copied through `nst` stages of LDS at
// `lds`.  Rows >= T and pieces past the end of a row count as zero: they are copied from valid addresses, or not at all, and
// zeroed when they are read.  TWO: the instruction's own sums are of at most kColsSteps steps, and are added up outside it:
// over waves as long as a shared launch has them its roundings go to one side (bf16, three layers of 16 positions, 4608 -> 512,
// and three of 64, 2304 -> 256: norms 7.8e-8 off in the mean, 1.1e-7 rms; so 6e-9 and 4.5e-8, for 4 % of the time).
template <int NB, int DT, bool TWO>
__device__ __forceinline__ void gram_cols_run(const unsigned char* __restrict__ X, int T, int row_bytes, int kb, int ke, int lane,
                                              unsigned char* lds, int nst, f32x16 (&total)[NB * (NB + 1) / 2]) {
    constexpr int NT = NB * (NB + 1) / 2;
    constexpr int COPIES = NB * 4;                       // copy instructions of a whole stage, 8 rows each
    const int n_stages = (ke - kb + kStageSteps - 1) / kStageSteps;
    const int copies = min(COPIES, (T + 7) / 8);         // those with rows inside the example
    const int limit = min(ke * 32, row_bytes);           // bytes of a row that this range has
    // chunk c (16 bytes) of a stage row r lies at position c ^ ((r >> 1) & 7): 16 rows read at one c meet no bank twice
    const unsigned char* src[COPIES];
    int at[COPIES];
#pragma unroll
    for (int i = 0; i < COPIES; ++i) {
        const int r = 8 * i + (lane >> 3);
        src[i] = X + (size_t)min(r, T - 1) * row_bytes;
        at[i] = kb * 32 + (((lane & 7) ^ ((r >> 1) & 7)) << 4);
    }
    const uint32_t base = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(LDS_PTR(unsigned char))lds);
    auto issue = [&](int buf) {                          // the next stage (inline assembly: waited for with wait_copies)
#pragma unroll
        for (int i = 0; i < COPIES; ++i) {
            if (i < copies) {
                const uint64_t from = (uint64_t)(uintptr_t)(src[i] + (at[i] < limit ? at[i] : 0));
                asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dwordx4 %1, off" :: "s"(base + (buf * copies + i) * 1024), "v"(from) : "memory", "m0");
            }
            at[i] += 128;
        }
    };
    const int row = lane & 31, half = lane >> 5;
    bool in[NB];
    uint32_t rd[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const int r = min(b * 32 + row, T - 1);
        in[b] = b * 32 + row < T;
        rd[b] = (uint32_t)(r * 128 + ((half ^ ((r >> 1) & 7)) << 4));
    }
    f32x16 chain[TWO ? NT : 1];
#pragma unroll
    for (int p = 0; p < (NB == 1 ? kStages1 : kStages2); ++p)
        if (p < nst && p < n_stages) issue(p);
    int buf = 0;
    for (int st = 0; st < n_stages; ++st) {
        wait_copies(min(n_stages - 1 - st, nst - 1) * copies);
        const unsigned char* sb = lds + buf * copies * 1024;
        uint4 f[kStageSteps][NB];
#pragma unroll
        for (int u = 0; u < kStageSteps; ++u)
#pragma unroll
            for (int b = 0; b < NB; ++b) f[u][b] = *reinterpret_cast<const uint4*>(sb + (rd[b] ^ (u << 5)));
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");          // read: the buffer takes a later stage
        if (st + nst < n_stages) issue(buf);
        buf = buf + 1 == nst ? 0 : buf + 1;
        const int k = kb + st * kStageSteps;
#pragma unroll
        for (int u = 0; u < kStageSteps; ++u) {
            if (k + u >= ke) break;                                  // uniform
            uint4 g[NB];
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const bool keep = in[b] && (k + u) * 32 + half * 16 < row_bytes;
                g[b] = make_uint4(keep ? f[u][b].x : 0u, keep ? f[u][b].y : 0u, keep ? f[u][b].z : 0u, keep ? f[u][b].w : 0u);
            }
            if constexpr (!TWO)            gram_cols_mfma<NB, DT>(g, total);
            else if (u == 0 && !(st & 1))  gram_cols_mfma<NB, DT, true>(g, chain);
            else                           gram_cols_mfma<NB, DT>(g, chain);
        }
        if constexpr (TWO) {
            static_assert(kColsSteps == 2 * kStageSteps, "");
            if ((st & 1) || st + 1 == n_stages) {
                if (st <= 1) {                                       // (total is zero: nothing to wait for)
#pragma unroll
                    for (int t = 0; t < NT; ++t) total[t] = chain[t];
                } else {
#pragma unroll
                    for (int t = 0; t < NT; ++t) total[t] += chain[t];
                }
            }
        }
    }
}

// float32 rows straight to registers, a lane's pieces of 8 steps in flight together.  VEC: rows of whole 16-byte pieces; else
// rows start at any 4-byte address, and a piece is four clamped 4-byte loads.
template <int NB, bool VEC>
__device__ __forceinline__ void gram_cols_run_loads(const float* __restrict__ X, int T, int D, int kb, int ke, int lane,
                                                    f32x16 (&acc)[NB * (NB + 1) / 2]) {
    const int row = lane & 31, half = lane >> 5;
    const float* p[NB];
    bool in[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const int r = b * 32 + row;
        in[b] = r < T;
        p[b] = X + (size_t)(r < T ? r : T - 1) * D;
    }
    for (int k = kb; k < ke; k += kColsSteps) {
        uint4 f[kColsSteps][NB];
#pragma unroll
        for (int u = 0; u < kColsSteps; ++u) {
            const int col = (k + u) * 8 + half * 4;
            const bool ok = (k + u) < ke && col < D;
            const int c = ok ? col : 0;
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const bool keep = ok && in[b];
                if (VEC) {
                    const uint4 v = *reinterpret_cast<const uint4*>(p[b] + c);
                    f[u][b] = make_uint4(keep ? v.x : 0u, keep ? v.y : 0u, keep ? v.z : 0u, keep ? v.w : 0u);
                } else {
                    const float x = p[b][c], y = p[b][min(c + 1, D - 1)], z = p[b][min(c + 2, D - 1)], w = p[b][min(c + 3, D - 1)];
                    f[u][b] = make_uint4(keep ? __float_as_uint(x) : 0u, (keep && c + 1 < D) ? __float_as_uint(y) : 0u,
                                         (keep && c + 2 < D) ? __float_as_uint(z) : 0u, (keep && c + 3 < D) ? __float_as_uint(w) : 0u);
                }
            }
        }
#pragma unroll
        for (int u = 0; u < kColsSteps; ++u) {
            if (k + u >= ke) break;                                  // uniform: the steps past the range hold zeros
            gram_cols_mfma<NB, 0>(f[u], acc);
        }
    }
}

// One workgroup's share.  run(X of the example, its columns, first step, end, sums): adds a range of steps of A or G.
template <int NB, typename Run>
__device__ __forceinline__ void gram_cols_block(const GramColsLayer& a, int item, float* part, unsigned char* lds, Run run) {
    constexpr int NT = NB * (NB + 1) / 2;            // tiles of the upper triangle
    constexpr int SHARE = 2 * NT * 4 * 64;           // 16-byte units of one wave's share (both products)
    const int ex = item / a.W, w = item - ex * a.W;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

    f32x16 acc[2][NT];
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[q][t][r] = 0.f;

    const int k0 = (w * 4 + wave) * a.per_wave;
    const int k1 = min(k0 + a.per_wave, a.steps);
    if (k0 < a.steps_a) run(a.A, (size_t)ex, a.d_in, k0, min(k1, a.steps_a), acc[0]);
    if (k1 > a.steps_a) run(a.G, (size_t)ex, a.d_out, max(k0, a.steps_a) - a.steps_a, k1 - a.steps_a, acc[1]);

    // waves 2, 3 -> LDS; waves 0, 1 add them; wave 1 -> LDS; wave 0 adds it and stores the workgroup's share
    auto put = [&](float4* slot) {
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    slot[((q * NT + t) * 4 + r) * 64 + lane] = make_float4(acc[q][t][4 * r], acc[q][t][4 * r + 1], acc[q][t][4 * r + 2], acc[q][t][4 * r + 3]);
    };
    auto add = [&](const float4* slot) {
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float4 v = slot[((q * NT + t) * 4 + r) * 64 + lane];
                    acc[q][t][4 * r] += v.x; acc[q][t][4 * r + 1] += v.y; acc[q][t][4 * r + 2] += v.z; acc[q][t][4 * r + 3] += v.w;
                }
    };
    float4* red = reinterpret_cast<float4*>(lds);
    __syncthreads();                                 // every wave is done with its stages
    if (wave >= 2) put(red + (wave - 2) * SHARE);
    __syncthreads();
    if (wave < 2) add(red + wave * SHARE);
    __syncthreads();
    if (wave == 1) put(red);
    __syncthreads();
    if (wave == 0) {
        add(red);
        put(reinterpret_cast<float4*>(part + a.part_off) + (size_t)item * SHARE);
    }
}

template <int NB, int DT, bool TWO, int CAP>
__device__ __forceinline__ void gram_cols_copied(const GramColsLayer& a, const GramColsArgs<CAP>& j, unsigned char* lds) {
    constexpr int ES = DT == 0 ? 4 : 2;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    gram_cols_block<NB>(a, blockIdx.x - a.first_block, j.part, lds,
        [&](const void* X, size_t ex, int D, int kb, int ke, f32x16 (&acc)[NB * (NB + 1) / 2]) {
            gram_cols_run<NB, DT, TWO>(static_cast<const unsigned char*>(X) + ex * a.T * D * ES, a.T, D * ES, kb, ke, lane,
                                       lds + wave * j.wave_lds, NB == 1 ? j.stages : kStages2, acc);
        });
}

// Rows of whole 16-byte pieces.  NB: the launch's largest number of 32-row blocks.  A layer alone may have more workgroups than
// two per compute unit: for three of them 168 registers (and no more LDS than the rows that there are).  (With the registers
// and the 64 KB of the kernel for several layers it lost 10 to 20 %: 60 examples of 8 positions, 5312 -> 2048, 10.9 and 13.5
// us, 174 of 20 positions, 1456 -> 528, 10.5 and 12.7.)
template <int NB, int DT, int CAP>
__global__ __launch_bounds__(kThreads, CAP == 1 ? 3 : 2) void k_gram_cols(GramColsArgs<CAP> j) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
    int li = 0;
    while (li + 1 < j.n_layers && blockIdx.x >= j.layer[li + 1].first_block) ++li;
    const GramColsLayer& a = j.layer[li];
    if constexpr (CAP == 1) {
        gram_cols_copied<NB, DT, false>(a, j, lds);
    } else {
        if (NB == 1 || a.nb == 1) gram_cols_copied<1, DT, true>(a, j, lds);
        else                      gram_cols_copied<NB, DT, true>(a, j, lds);
    }
}

// float32 rows of any length, through registers
template <int NB, int CAP>
__global__ __launch_bounds__(kThreads, 2) void k_gram_cols_loads(GramColsArgs<CAP> j) {
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
    int li = 0;
    while (li + 1 < j.n_layers && blockIdx.x >= j.layer[li + 1].first_block) ++li;
    const GramColsLayer& a = j.layer[li];
    const int lane = threadIdx.x & 63;
    gram_cols_block<NB>(a, blockIdx.x - a.first_block, j.part, lds,
        [&](const void* X, size_t ex, int D, int kb, int ke, f32x16 (&acc)[NB * (NB + 1) / 2]) {
            const float* x = static_cast<const float*>(X) + ex * a.T * D;
            // (the choice sits outside the loops: a branch around every load would make each wait for the one before)
            if ((D & 3) == 0) gram_cols_run_loads<NB, true>(x, a.T, D, kb, ke, lane, acc);
            else              gram_cols_run_loads<NB, false>(x, a.T, D, kb, ke, lane, acc);
        });
}

// Several layers: sums[ex][t] of a layer = the sum over the entries of triangle tile t of (sum_w P_w) * (sum_w Q_w), the
// tile (0,1) counted twice (it stands for its mirror image too), the shares added in the order of the workgroups.  One
// workgroup per (example, tile).  (A workgroup per example that walked all layers' shares read them at 20 GB/s each: 13 and
// 19 us for 32 examples of four layers.)
__global__ __launch_bounds__(kThreads) void k_gram_cols_sums(GramColsArgs<kGramColsLayers> j) {
    __shared__ float red[4];
    int li = 0;
    while (li + 1 < j.n_layers && blockIdx.x >= j.layer[li + 1].first_finish) ++li;
    const GramColsLayer& a = j.layer[li];
    const int nt = a.nb == 1 ? 1 : 3, item = blockIdx.x - a.first_finish;
    const int ex = item / nt, t = item - ex * nt;
    const float4* base = reinterpret_cast<const float4*>(j.part + a.part_off) + ((size_t)ex * a.W * 2 * nt + t) * kThreads + threadIdx.x;
    float4 p = make_float4(0.f, 0.f, 0.f, 0.f), q = p;
    auto sum = [](float4& x, const float4& y) { x.x += y.x; x.y += y.y; x.z += y.z; x.w += y.w; };
#pragma unroll 4
    for (int w = 0; w < a.W; ++w) {
        sum(p, base[(size_t)w * 2 * nt * kThreads]);
        sum(q, base[((size_t)w * 2 + 1) * nt * kThreads]);
    }
    float s = (p.x * q.x + p.y * q.y) + (p.z * q.z + p.w * q.w);
    s = block_sum_256(s, red);
    if (threadIdx.x == 0) a.sums[item] = (nt == 3 && t == 1) ? 2.0f * s : s;
}

// The same added up, sqnorm[ex] (+)=, where no other layer's sums are to be added: one launch less.  One workgroup of 1024
// threads per example, an entry of every tile a thread.  (A tile per quarter of the threads, 16 bytes at a time, took twice as
// long: two layers of 62 positions, 15 and 4 shares, 11 and 21 us.)
constexpr int kFinishThreads = 1024;
template <int NT>
__device__ __forceinline__ float gram_cols_dot(const float* base, int W) {
    constexpr int HALF = NT * 16 * 64;
    float p[NT], q[NT];
#pragma unroll
    for (int i = 0; i < NT; ++i) { p[i] = 0.f; q[i] = 0.f; }
#pragma unroll 4
    for (int w = 0; w < W; ++w) {
#pragma unroll
        for (int i = 0; i < NT; ++i) {
            p[i] += base[(size_t)w * 2 * HALF + i * kFinishThreads];
            q[i] += base[(size_t)w * 2 * HALF + HALF + i * kFinishThreads];
        }
    }
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < NT; ++i) s += (NT == 3 && i == 1) ? 2.0f * (p[i] * q[i]) : p[i] * q[i];
    return s;
}
template <int CAP>
__global__ __launch_bounds__(kFinishThreads) void k_gram_cols_finish(GramColsArgs<CAP> j, int accumulate, float* __restrict__ sqnorm, float C,
                                                                       float* __restrict__ clip) {
    __shared__ float red[kFinishThreads / 64];
    const int ex = blockIdx.x;
    float s = 0.f;
    for (int li = 0; li < j.n_layers; ++li) {
        const GramColsLayer& a = j.layer[li];
        const float* base = j.part + a.part_off + threadIdx.x;
        if (a.nb == 1) s += gram_cols_dot<1>(base + (size_t)ex * a.W * 2 * 1024, a.W);
        else           s += gram_cols_dot<3>(base + (size_t)ex * a.W * 2 * 3072, a.W);
    }
    s = wave_sum(s);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x >= 64) return;
    // (in a tree: one after the other these additions were most of a norm's error)
    const float v = wave_sum(threadIdx.x < kFinishThreads / 64 ? red[threadIdx.x] : 0.f);
    if (threadIdx.x == 0) {
        const float t = accumulate ? sqnorm[ex] + v : v;
        sqnorm[ex] = t;
        if (clip) clip[ex] = clip_factor_of(t, C);
    }
}

}  // namespace

GramColsPlan plan_gram_cols(int B, int T, int d_in, int d_out, int dt) {
    GramColsPlan p{};
    const int piece = dt == 0 ? 4 : 8;                   // columns of a 16-byte piece; a step is two pieces
    if (B < 1 || T < 2 || T > 64 || dt < 0 || dt > 2 || d_in < 1 || d_out < 1) return p;
    if (dt != 0 && ((d_in | d_out) % piece) != 0) return p;     // 16-bit rows: whole 16-byte pieces only
    const int steps = ceil_div(d_in, 2 * piece) + ceil_div(d_out, 2 * piece);
    // fill the chip (2 workgroups on each of 256 compute units) with waves of at least kColsSteps steps
    int W = ceil_div(512, B);
    const int w_max = steps / (4 * kColsSteps);
    if (W > w_max) W = w_max;
    if (W > 64) W = 64;
    if (W < 2) return p;                                 // enough examples, or rows too narrow to split
    p.use = true;
    p.nb = T <= 32 ? 1 : 2;
    p.per_wave = ceil_div(steps, 4 * W);
    p.W = ceil_div(steps, 4 * p.per_wave);               // no workgroup without a step
    const int nt = p.nb * (p.nb + 1) / 2;
    p.ws_floats = (size_t)B * p.W * 2 * nt * 16 * 64;
    return p;
}

int gram_cols_sums(const GramColsPlan& p) { return p.nb == 1 ? 1 : 3; }

int gram_cols_kind(int T, int d_in, int d_out, int dt) {
    return dt != 0 || ((d_in | d_out) & 3) == 0 ? 0 : T <= 32 ? 1 : 2;
}

namespace {
// the kind of a launch: that of the layers that have one
int cols_launch_kind(const GramLayerDesc* layers, int n_layers, int dt) {
    int kind = 0;
    for (int l = 0; l < n_layers; ++l) kind = std::max(kind, gram_cols_kind(layers[l].T, layers[l].d_in, layers[l].d_out, dt));
    return kind;
}

// The layers of a shared launch fill the chip together, so each takes fewer workgroups than it would alone, all of about one
// length: few shares to store and to add, and waves that stream (a wave of kColsSteps waits once for all it loads).  The
// length, counted in steps of 32 rows, that makes  rounds of 512 workgroups x (length + what a workgroup costs besides)
// least, of those whose shares take at most max_floats (at the longest, one workgroup per example, they do).  A layer alone,
// and those that are loaded 4 bytes at a time, a memory round trip for 8 steps, keep their own plans where those fit (49
// examples of 17 positions, 656 -> 1673 and 1673 -> 656 among four layers: 19 us, 30 us with long waves).
void plan_cols_shared(const GramLayerDesc* layers, int n_layers, int B, int dt, size_t max_floats, GramColsPlan* p) {
    constexpr int kOverhead = 24;
    const int step = dt == 0 ? 8 : 16;
    int steps[kGramColsLayers], longest = kColsSteps;
    size_t own = 0;
    for (int l = 0; l < n_layers; ++l) {
        p[l] = plan_gram_cols(B, layers[l].T, layers[l].d_in, layers[l].d_out, dt);
        steps[l] = ceil_div(layers[l].d_in, step) + ceil_div(layers[l].d_out, step);
        longest = longest > p[l].nb * ceil_div(steps[l], 4) ? longest : p[l].nb * ceil_div(steps[l], 4);
        own += p[l].ws_floats;
    }
    if ((n_layers == 1 || cols_launch_kind(layers, n_layers, dt) != 0) && own <= max_floats) return;
    auto take = [&](int l, int length, int& W) {              // whole stages per wave, so that the copies move whole lines
        const int least = length / p[l].nb > kColsSteps ? length / p[l].nb : kColsSteps;
        const int w = ceil_div(steps[l], 4 * least);
        const int per_wave = (ceil_div(steps[l], 4 * w) + kStageSteps - 1) / kStageSteps * kStageSteps;
        W = ceil_div(steps[l], 4 * per_wave);
        return per_wave;
    };
    int64_t best_cost = -1;
    int best = longest;
    for (int length = kColsSteps; length < longest + 16; length += length < 64 ? 4 : 16) {
        const int len = length < longest ? length : longest;
        int64_t blocks = 0;
        int most = 0;
        size_t floats = 0;
        for (int l = 0; l < n_layers; ++l) {
            int W;
            const int per_wave = take(l, len, W);
            blocks += (int64_t)B * W;
            floats += p[l].ws_floats / (size_t)p[l].W * (size_t)W;
            most = most > p[l].nb * per_wave ? most : p[l].nb * per_wave;
        }
        if (floats > max_floats) continue;
        const int64_t cost = ((blocks + 511) / 512) * (most + kOverhead);
        if (best_cost < 0 || cost < best_cost) { best_cost = cost; best = len; }
        if (blocks <= 512) break;                             // one round: longer waves only take longer
    }
    for (int l = 0; l < n_layers; ++l) {
        const size_t share = p[l].ws_floats / (size_t)p[l].W;
        p[l].per_wave = take(l, best, p[l].W);
        p[l].ws_floats = share * (size_t)p[l].W;
    }
}

template <int NB, int CAP> void launch_cols_copied(unsigned blocks, size_t lds, hipStream_t st, int dt, const GramColsArgs<CAP>& a) {
    if (dt == 0)      k_gram_cols<NB, 0, CAP><<<blocks, kThreads, lds, st>>>(a);
    else if (dt == 1) k_gram_cols<NB, 1, CAP><<<blocks, kThreads, lds, st>>>(a);
    else              k_gram_cols<NB, 2, CAP><<<blocks, kThreads, lds, st>>>(a);
}

// fills the launch's arguments and makes the first launch; sums: nullptr, or each layer's own array
template <int CAP>
hipError_t launch_cols(const GramLayerDesc* layers, float* const* sums, int n_layers, int B, float* ws, size_t max_floats, hipStream_t st, int dt,
                       GramColsArgs<CAP>& a, unsigned& finish_blocks) {
    if (n_layers < 1 || n_layers > CAP || dt < 0 || dt > 2) return hipErrorInvalidValue;
    a.part = ws; a.n_layers = n_layers;
    const int step = dt == 0 ? 8 : 16;
    const int kind = cols_launch_kind(layers, n_layers, dt);
    int64_t blocks = 0, finish = 0;
    size_t off = 0;
    int nb = 1, rows = 0;
    GramColsPlan plans[CAP];
    plan_cols_shared(layers, n_layers, B, dt, max_floats, plans);
    for (int l = 0; l < n_layers; ++l) {
        const GramLayerDesc& y = layers[l];
        const GramColsPlan& p = plans[l];
        if (!p.use || (kind != 0 && p.nb != kind)) return hipErrorInvalidValue;
        GramColsLayer& g = a.layer[l];
        g.A = y.A; g.G = y.G;
        g.sums = sums ? sums[l] : nullptr;
        g.part_off = off;
        g.T = y.T; g.d_in = y.d_in; g.d_out = y.d_out;
        g.steps_a = ceil_div(y.d_in, step); g.steps = g.steps_a + ceil_div(y.d_out, step);
        g.W = p.W; g.per_wave = p.per_wave; g.nb = p.nb;
        g.first_block = (unsigned)blocks; g.first_finish = (unsigned)finish;
        blocks += (int64_t)B * p.W;
        finish += (int64_t)B * gram_cols_sums(p);
        off += p.ws_floats;
        nb = std::max(nb, p.nb); rows = std::max(rows, y.T);
    }
    for (int l = n_layers; l < CAP; ++l) a.layer[l] = a.layer[0];
    if (blocks >= (int64_t(1) << 24) || finish >= (int64_t(1) << 24)) return hipErrorInvalidValue;   // (W >= 2 only where B < 2^9)
    finish_blocks = (unsigned)finish;
    // where a workgroup's shares meet: two waves' sums of both products, the tiles of one 32-row block or of two
    const int meet = nb == 1 ? 16384 : 3 * 16384;
    // Rows that are no whole 16-byte pieces are loaded to registers: what hides their many short loads is the number of
    // workgroups (with the copied layers in one launch, two per compute unit, two layers of 64 examples lost half: 20 positions,
    // 662 -> 600, and 41, 367 -> 3519, 49 and 104 us).  So is a float32 layer alone where three workgroups of 48 KB fill the
    // chip and two of 64 KB would leave a second round (174 examples of 64 positions, 1456 -> 528: 41 and 46 us; 16 bits, half
    // the products, gain from whole lines there too).
    if (kind != 0 || (CAP == 1 && dt == 0 && layers[0].T > 48 && blocks > 512 && blocks <= 768)) {
        if (nb == 1) k_gram_cols_loads<1, CAP><<<(unsigned)blocks, kThreads, (size_t)meet, st>>>(a);
        else         k_gram_cols_loads<2, CAP><<<(unsigned)blocks, kThreads, (size_t)meet, st>>>(a);
        return hipGetLastError();
    }
    a.stages = kStages1; a.wave_lds = kWaveLds;
    if (CAP == 1 || nb == 1) {
        // no more LDS than the rows that there are, and fewer stages in flight where a compute unit has more than two workgroups
        const int stage = ceil_div(rows, 8) * 1024, per_cu = (int)((blocks + 255) / 256);
        while (a.stages > 2 && std::max(meet, 4 * a.stages * stage) * per_cu > 160 * 1024) --a.stages;
        a.wave_lds = (nb == 1 ? a.stages : kStages2) * stage;
    }
    const size_t lds = (size_t)std::max(meet, 4 * a.wave_lds);
    if (nb == 1) launch_cols_copied<1, CAP>((unsigned)blocks, lds, st, dt, a);
    else         launch_cols_copied<2, CAP>((unsigned)blocks, lds, st, dt, a);
    return hipGetLastError();
}

template <int CAP>
hipError_t launch_cols_norms(const GramLayerDesc* layers, int n_layers, int B, bool accumulate, float* sqnorm, float* ws, size_t max_floats, hipStream_t st,
                             int dt, const ClipOut* co) {
    GramColsArgs<CAP> a;
    unsigned finish = 0;
    const hipError_t e = launch_cols<CAP>(layers, nullptr, n_layers, B, ws, max_floats, st, dt, a, finish);
    if (e != hipSuccess) return e;
    k_gram_cols_finish<CAP><<<B, kFinishThreads, 0, st>>>(a, accumulate ? 1 : 0, sqnorm, co ? co->C : 0.f, co ? co->clip : nullptr);
    return hipGetLastError();
}
}  // namespace

hipError_t launch_gram_cols_layers(const GramLayerDesc* layers, float* const* sums, int n_layers, int B, float* ws, size_t max_floats,
                                   hipStream_t st, int dt) {
    GramColsArgs<kGramColsLayers> a;
    unsigned finish = 0;
    const hipError_t e = launch_cols<kGramColsLayers>(layers, sums, n_layers, B, ws, max_floats, st, dt, a, finish);
    if (e != hipSuccess) return e;
    k_gram_cols_sums<<<finish, kThreads, 0, st>>>(a);
    return hipGetLastError();
}

hipError_t launch_gram_cols_norms(const GramLayerDesc* layers, int n_layers, int B, bool accumulate, float* sqnorm, float* ws, size_t max_floats,
                                  hipStream_t st, int dt, const ClipOut* co) {
    if (n_layers == 1) return launch_cols_norms<1>(layers, 1, B, accumulate, sqnorm, ws, max_floats, st, dt, co);
    return launch_cols_norms<kGramColsLayers>(layers, n_layers, B, accumulate, sqnorm, ws, max_floats, st, dt, co);
}

hipError_t launch_gram_cols(const GramColsPlan& p, const void* A, const void* G, int B, int T, int d_in, int d_out,
                            bool accumulate, float* sqnorm, float* ws, hipStream_t st, int dt, const ClipOut* co) {
    if (!p.use) return hipErrorInvalidValue;
    const GramLayerDesc y{A, G, T, d_in, d_out, nullptr, nullptr};
    return launch_gram_cols_norms(&y, 1, B, accumulate, sqnorm, ws, kAnySlices, st, dt, co);
}

}  // namespace dpk
