// Gram path of the per-example squared norm for float32 inputs:
//     ||A_i^T G_i||_F^2 = sum_{t,s} (A_i A_i^T)_{ts} (G_i G_i^T)_{ts}.
// Same decomposition as the 16-bit Gram kernels: one workgroup per example and pair of row tiles (t-tile <= s-tile),
// the tile of A_i A_i^T (contraction over d_in) and then the tile of G_i G_i^T (contraction over d_out) kept in MFMA
// accumulators of identical layout, multiplied lane by lane and reduced; off-diagonal pairs count twice, and so does the
// upper right quarter of a diagonal tile, whose mirror image is not computed.
// The products run on the bf16 MFMA with every operand split into three bf16 numbers (dp_split.h): the rate of the fp32
// MFMA (157 TFLOP/s nominal) bounded them, six bf16 products have 2.7 times that.  Each element is split once, on its
// way into LDS: stages of 16 columns, two in LDS, the loads of two stages at a time (whole 128-byte lines of the rows)
// wait in registers; a thread's four columns are half an MFMA operand of 8, 8 bytes per part.
#include <algorithm>
#include "dp_common.h"
#include "dp_internal.h"
#include "dp_split.h"

namespace dpk {

namespace {

struct GramF32Layer {
    const float* A;
    const float* G;
    float* partial;      // [B][npairs]
    int T, d_in, d_out, npairs, n_items;
    int first_item;      // among the items of one XCD
};
struct GramF32Args {
    GramF32Layer layer[kJointLayers];
    int n_layers;
};

constexpr int GK = 16;        // contraction elements per stage: one MFMA deep

// MI: 32-row blocks per wave and side; the tile has 64 MI rows
template <int MI> struct GramTile {
    static constexpr int R = 64 * MI;
    static constexpr int PLANE = R * 16 + 64;              // bytes of [8 columns of a part][row]; the 64 bytes keep the two halves of a write in different banks
    static constexpr int SIDE = 6 * PLANE;                 // [part][k / 8]
    static constexpr int STAGE = 2 * SIDE;                 // rows of the t-tile, rows of the s-tile
};

// The wave's tile of X_t X_s^T once more with the float32 instruction, in the order of k, straight from memory and slow:
// for sums of 2^80 and more, infinities and NaN (see dp_split.h).
template <int MI>
__device__ __forceinline__ void gram_f32_exact(const float* Xi, int T, int D, int t0, int s0, f32x16 (&acc)[MI][MI]) {
    const int lrow = threadIdx.x & 31, lhalf = (threadIdx.x & 63) >> 5;
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < MI; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    for (int k = 0; k < D; k += 2) {
        const bool in = k + lhalf < D;
        const int c = in ? k + lhalf : 0;
        float ft[MI], fs[MI];
#pragma unroll
        for (int i = 0; i < MI; ++i) {
            const int rt = t0 + 32 * i + lrow, rs = s0 + 32 * i + lrow;
            const float xt = Xi[(size_t)min(rt, T - 1) * D + c], xs = Xi[(size_t)min(rs, T - 1) * D + c];
            ft[i] = in && rt < T ? xt : 0.f;
            fs[i] = in && rs < T ? xs : 0.f;
        }
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < MI; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(ft[i], fs[j], acc[i][j], 0, 0, 0);
    }
}

// One Gram product tile: acc = X[t-tile rows] . X[s-tile rows]^T over the D columns of X_i[T, D].
// LOAD: how a thread's four columns come: 2 = one 16-byte buffer load (D % 4 == 0: every such piece lies inside a row or
// outside it), 1 = four 4-byte buffer loads, 0 = four loads by address (D >= 2^22: a tile's rows span 2^31 bytes or more).
// Every wave leaves with its LDS reads done.
template <int MI, int LOAD, bool DIAG>
__device__ __forceinline__ void gram_f32_product(const float* __restrict__ Xi, int T, int D, int t0, int s0,
                                                 unsigned char* lds, f32x16 (&acc)[MI][MI]) {
    using GT = GramTile<MI>;
    constexpr int SIDES = DIAG ? 1 : 2;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave >> 1, wn = wave & 1;
    const int lrow = lane & 31, lhalf = lane >> 5;
    // global -> LDS: four threads per row, MI rows of either side and two stages (a 128-byte line of the row) at a time
    const int lr = tid >> 2, lc = (tid & 3) * 4;
    const int t_rows = min(T - t0, GT::R), s_rows = min(T - s0, GT::R);
    // buffer loads: a row past T or a column past D lies outside the buffer and comes back as zero
    const auto buf_t = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(Xi + (size_t)t0 * D), (short)0, LOAD ? t_rows * D * 4 : 0, 0x00020000);
    const auto buf_s = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(Xi + (size_t)s0 * D), (short)0, LOAD ? s_rows * D * 4 : 0, 0x00020000);
    const uint32_t wr = (uint32_t)((lc >> 3) * GT::PLANE + lr * 16 + (lc & 4) * 2);
    f32x4 x[2][SIDES][MI];
    int next_k = lc;
    auto fetch = [&]() {
#pragma unroll
        for (int h = 0; h < SIDES; ++h)
#pragma unroll
            for (int v = 0; v < MI; ++v)
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const int row = lr + 64 * v, k = next_k + u * GK;
                    if (LOAD == 2) {
                        const uint32_t off = k < D ? (uint32_t)(row * D + k) * 4u : 0x7ffffff0u;
                        x[u][h][v] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(h == 0 ? buf_t : buf_s, off, 0, 0));
                    } else if (LOAD == 1) {
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            const uint32_t off = k + j < D ? (uint32_t)(row * D + k + j) * 4u : 0x7ffffff0u;
                            x[u][h][v][j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(h == 0 ? buf_t : buf_s, off, 0, 0));
                        }
                    } else {
                        const bool in = row < (h == 0 ? t_rows : s_rows);
                        const float* p = Xi + (size_t)((h == 0 ? t0 : s0) + (in ? row : 0)) * D;
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            const float q = p[k + j < D ? k + j : 0];
                            x[u][h][v][j] = in && k + j < D ? q : 0.f;
                        }
                    }
                }
        next_k += 2 * GK;
    };
    // the split of one of the thread's SIDES * MI pieces of stage half u
    auto split_step = [&](int u, int piece, int buf) {
        const int h = piece / MI, v = piece % MI;
        uint32_t part[3][2];
#pragma unroll
        for (int q = 0; q < 2; ++q)
            split2(x[u][h][v][2 * q] * kSplitScale, x[u][h][v][2 * q + 1] * kSplitScale, part[0][q], part[1][q], part[2][q]);
#pragma unroll
        for (int p = 0; p < 3; ++p)
            *reinterpret_cast<uint2*>(lds + buf * GT::STAGE + h * GT::SIDE + p * 2 * GT::PLANE + wr + v * 64 * 16) =
                make_uint2(part[p][0], part[p][1]);
    };
    const uint32_t rdT = (uint32_t)(lhalf * GT::PLANE + (wm * MI * 32 + lrow) * 16);
    const uint32_t rdS = (uint32_t)((DIAG ? 0 : GT::SIDE) + lhalf * GT::PLANE + (wn * MI * 32 + lrow) * 16);
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < MI; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    constexpr int TILES = MI * MI, PIECES = SIDES * MI, STEPS = (PIECES + TILES - 1) / TILES;
    fetch();
#pragma unroll
    for (int q = 0; q < PIECES; ++q) split_step(0, q, 0);
    __builtin_amdgcn_s_waitcnt(0xC07F);
    __builtin_amdgcn_s_barrier();
    // Past the last column the copies bring zeros: the loop takes two stages a turn and has no branches.  One 32 x 32 tile
    // of the wave after the other: its six MFMAs, in their shadow a share of the next stage's split and the addition of
    // the tile before.  The idle wave of a diagonal pair multiplies as well and drops its sums below (a branch around
    // its MFMAs would end the interleaving for all).
    f32x16 pend = {};                                      // the sums of the tile before, not yet added
    for (int k0 = 0; k0 < D; k0 += 2 * GK) {
#pragma unroll
        for (int buf = 0; buf < 2; ++buf) {
            bf16x8 ft[MI][3], fs[MI][3];
            const unsigned char* sb = lds + buf * GT::STAGE;
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int p = 0; p < 3; ++p) {
                    ft[i][p] = *reinterpret_cast<const bf16x8*>(sb + rdT + p * 2 * GT::PLANE + i * 512);
                    fs[i][p] = *reinterpret_cast<const bf16x8*>(sb + rdS + p * 2 * GT::PLANE + i * 512);
                }
#pragma unroll
            for (int t = 0; t < TILES; ++t) {
                const int before = (t + TILES - 1) % TILES;
                acc[before / MI][before % MI] += pend * kSplitUnscale;
                pend = split_mfma(ft[t / MI], fs[t % MI]);
#pragma unroll
                for (int q = 0; q < STEPS; ++q)
                    if (t * STEPS + q < PIECES) split_step(buf ^ 1, t * STEPS + q, buf ^ 1);
                if (t == TILES - 1 && buf == 0) fetch();
#pragma unroll
                for (int q = 0; q < 6; ++q) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x002, 7, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            __builtin_amdgcn_s_waitcnt(0xC07F);            // lgkmcnt(0): this wave's parts of the next stage are in LDS
            __builtin_amdgcn_s_barrier();
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    acc[MI - 1][MI - 1] += pend * kSplitUnscale;
    SplitCheck check;
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < MI; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) check.add(acc[i][j][r]);
    if (__any(check.suspect())) gram_f32_exact<MI>(Xi, T, D, t0 + wm * MI * 32, s0 + wn * MI * 32, acc);
}

template <int MI, int LOAD, bool DIAG>
__device__ __forceinline__ void gram_f32_pair(const GramF32Layer& a, int ex, int tt, int ss, unsigned char* lds, float* out) {
    constexpr int R = GramTile<MI>::R;
    f32x16 accP[MI][MI], accQ[MI][MI];
    gram_f32_product<MI, LOAD, DIAG>(a.A + (size_t)ex * a.T * a.d_in, a.T, a.d_in, tt * R, ss * R, lds, accP);
    gram_f32_product<MI, LOAD, DIAG>(a.G + (size_t)ex * a.T * a.d_out, a.T, a.d_out, tt * R, ss * R, lds, accQ);
    // rows beyond T were stored as zeros, so their entries of both tiles are zero
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < MI; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) s += accP[i][j][r] * accQ[i][j][r];
    if (DIAG && (threadIdx.x >> 6) == 1) s += s;            // wave 2 holds the mirror image of wave 1's quarter
    if (DIAG && (threadIdx.x >> 6) == 2) s = 0.f;
    s = block_sum_256(s, reinterpret_cast<float*>(lds));
    if (threadIdx.x == 0) *out = DIAG ? s : 2.0f * s;
}

// Items (layer, example, tile pair), the layers in the order given.  Workgroup b runs on XCD b % 8: every XCD takes a
// contiguous eighth of every layer's items, example by example, so that an example's pairs read its rows through one L2
// and the XCDs have equal work (an eighth of the whole list gave those with the widest layer 1.25 times the mean: four
// layers of 768 .. 3072 columns, B = 64, T = 512: 1.71 ms, 1.39 ms so).
template <int MI, int LOAD>
__global__ __launch_bounds__(kThreads, MI == 2 ? 2 : 4) void k_gram_f32(GramF32Args g) {
    __shared__ __attribute__((aligned(1024))) unsigned char lds[2 * GramTile<MI>::STAGE];
    const int L = blockIdx.x >> 3;
    int l = 0;
    while (l + 1 < g.n_layers && L >= g.layer[l + 1].first_item) ++l;
    const GramF32Layer a = g.layer[l];
    const int item = (int)(blockIdx.x & 7) * ((a.n_items + 7) >> 3) + L - a.first_item;
    if (item >= a.n_items) return;
    const int ex = item / a.npairs, pair0 = item - ex * a.npairs;
    int pair = pair0;
    // pair -> (tt, ss), tt <= ss, rows of the upper triangle in order
    const int nt = (a.T + GramTile<MI>::R - 1) / GramTile<MI>::R;
    int tt = 0;
    while (pair >= nt - tt) { pair -= nt - tt; ++tt; }
    const int ss = tt + pair;
    float* out = a.partial + (size_t)ex * a.npairs + pair0;
    if (tt == ss) gram_f32_pair<MI, LOAD, true>(a, ex, tt, ss, lds, out);
    else          gram_f32_pair<MI, LOAD, false>(a, ex, tt, ss, lds, out);
}

struct GramArgsF {
    const float* A;
    const float* G;
    float* partial;      // [B][npairs]
    int T, d_in, d_out;
};

// Short sequences (T <= 32: the late convolutions of an image model, 16 positions of 2304 to 4608 inputs): the kernel
// above would give the one useful 32 x 32 tile to one wave, a chain of d / 2 dependent 64-cycle MFMAs (75 to 135 us
// for such layers), while three waves multiply zeros.  Here the four waves split the contraction: every stage holds
// 128 columns of the example's rows, wave w takes columns 32 w .. 32 w + 31 of it, and the four partial tiles are
// added through LDS in the order w = 0 .. 3, first for A A^T, then for G G^T; the tile is diagonal, so both MFMA
// operands are the same fragment.  One workgroup per example.
constexpr int SK = 128;       // contraction elements per stage
constexpr int SP = SK + 1;    // padded row length in LDS
template <bool VEC>
__device__ __forceinline__ void gram_small_product(const float* __restrict__ Xi, int T, int D, float (*sX)[SP],
                                                   float (*part)[32][33], float (*out)[33]) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int lrow = lane & 31, lhalf = lane >> 5;
    // global -> LDS: a thread moves four 4-column pieces per stage: rows lr + 8 v, columns lc .. lc + 3
    const int lr = tid >> 5, lc = (tid & 31) * 4;
    f32x16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;
    float x[2][4][4];
    auto fetch = [&](int b, int k0) {
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int row = lr + 8 * v;
            const float* p = Xi + (size_t)(row < T ? row : T - 1) * D;
            if (VEC) {
                const int c = (k0 + lc < D) ? k0 + lc : 0;
                const float4 q = *reinterpret_cast<const float4*>(p + c);
                x[b][v][0] = q.x; x[b][v][1] = q.y; x[b][v][2] = q.z; x[b][v][3] = q.w;
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j) x[b][v][j] = p[(k0 + lc + j < D) ? k0 + lc + j : 0];
            }
        }
    };
    auto commit = [&](int b, int k0) {
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                sX[lr + 8 * v][lc + j] = (lr + 8 * v < T && k0 + lc + j < D) ? x[b][v][j] : 0.f;
    };
    // two stages of loads in flight
    if (D > 0) fetch(0, 0);
    if (D > SK) fetch(1, SK);
    for (int k0 = 0; k0 < D; k0 += 2 * SK) {
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const int kb = k0 + b * SK;
            if (kb >= D) break;
            commit(b, kb);
            __syncthreads();
            if (kb + 2 * SK < D) fetch(b, kb + 2 * SK);
            float f[16];
#pragma unroll
            for (int j = 0; j < 16; ++j) f[j] = sX[lrow][wave * 32 + 2 * j + lhalf];
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int j = 0; j < 16; ++j) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(f[j], f[j], acc, 0, 0, 0);
            __syncthreads();
        }
    }
    // accumulator element r of a lane: row 8 (r / 4) + 4 lhalf + r % 4, column lrow
#pragma unroll
    for (int r = 0; r < 16; ++r) part[wave][8 * (r >> 2) + 4 * lhalf + (r & 3)][lrow] = acc[r];
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int idx = tid + 256 * e, mr = idx >> 5, nc = idx & 31;
        out[mr][nc] = ((part[0][mr][nc] + part[1][mr][nc]) + part[2][mr][nc]) + part[3][mr][nc];
    }
    __syncthreads();
}

template <bool VEC>
__global__ __launch_bounds__(kThreads) void k_gram_f32_small(GramArgsF a) {
    __shared__ float sX[32][SP];
    __shared__ float part[4][32][33];
    __shared__ float P[32][33], Q[32][33];
    __shared__ float red[4];
    const int ex = blockIdx.x;
    gram_small_product<VEC>(a.A + (size_t)ex * a.T * a.d_in, a.T, a.d_in, sX, part, P);
    gram_small_product<VEC>(a.G + (size_t)ex * a.T * a.d_out, a.T, a.d_out, sX, part, Q);
    // rows beyond T were stored as zeros, so their entries of both tiles are zero
    float s = 0.f;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int idx = threadIdx.x + 256 * e, mr = idx >> 5, nc = idx & 31;
        s += P[mr][nc] * Q[mr][nc];
    }
    s = block_sum_256(s, red);
    if (threadIdx.x == 0) a.partial[ex] = s;
}

}  // namespace

// Tiles of 64 or 128 rows.  In workgroups' time of the 128-row tile (two fit a compute unit, four of the 64-row one), an item
// of 64-row tiles takes 0.425 of it where the chip is full and 0.6 where it is not; 64-row tiles waste less of a sequence
// that is no multiple of 128 (B = 9, T = 192, 844 x 1664: 0.14 ms on them, 0.18 ms on 128-row tiles), 128-row tiles read
// their fragments half as often (B = 64, T = 512).  At most the pairs of 64-row tiles: gram_f32_sums.
GramPlan plan_gram_f32(int B, int T) {
    const auto pairs = [&](int tile) { const int64_t nt = (T + tile - 1) / tile; return nt * (nt + 1) / 2; };
    const double cost128 = std::max(0.5, (double)B * pairs(128) / 256), cost64 = std::max(0.3, 0.425 * B * pairs(64) / 256);
    GramPlan p;
    p.tile = T > 64 && cost128 <= cost64 ? 128 : 64;
    p.nt = (T + p.tile - 1) / p.tile;
    p.npairs = (int)pairs(p.tile);
    return p;
}

int gram_f32_sums(int T) { const int nt = (T + 63) / 64; return nt * (nt + 1) / 2; }

// 1 + the way of loading, + 3 for tiles of 128 rows
int gram_f32_class(int B, int T, int d_in, int d_out) {
    if (T <= 32) return 0;
    const int load = (d_in | d_out) >= (1 << 22) ? 0 : ((d_in | d_out) & 3) == 0 ? 2 : 1;
    return 1 + load + (plan_gram_f32(B, T).tile == 128 ? 3 : 0);
}

hipError_t launch_gram_f32_layers(const JointShape* sh, const JointOperands* op, float* const* partial, int n_layers, int B,
                                  hipStream_t st) {
    if (n_layers < 1 || n_layers > kJointLayers) return hipErrorInvalidValue;
    const int cls = gram_f32_class(B, sh[0].T, sh[0].M, sh[0].N);
    if (cls == 0) return hipErrorInvalidValue;
    GramF32Args g;
    int64_t first = 0;
    for (int l = 0; l < n_layers; ++l) {
        if (gram_f32_class(B, sh[l].T, sh[l].M, sh[l].N) != cls) return hipErrorInvalidValue;
        GramF32Layer& y = g.layer[l];
        y.A = reinterpret_cast<const float*>(op[l].A); y.G = reinterpret_cast<const float*>(op[l].G); y.partial = partial[l];
        y.T = sh[l].T; y.d_in = sh[l].M; y.d_out = sh[l].N;
        y.npairs = plan_gram_f32(B, sh[l].T).npairs;
        y.first_item = (int)first;
        const int64_t n = (int64_t)y.npairs * B;
        if (n >= (int64_t(1) << 31) - 8) return hipErrorInvalidValue;
        y.n_items = (int)n;
        first += (n + 7) / 8;
        if (!launch_holds(8 * first, kThreads)) return hipErrorInvalidValue;
    }
    for (int l = n_layers; l < kJointLayers; ++l) g.layer[l] = g.layer[0];
    g.n_layers = n_layers;
    const unsigned grid = 8u * (unsigned)first;
    if      (cls == 1) k_gram_f32<1, 0><<<grid, kThreads, 0, st>>>(g);
    else if (cls == 2) k_gram_f32<1, 1><<<grid, kThreads, 0, st>>>(g);
    else if (cls == 3) k_gram_f32<1, 2><<<grid, kThreads, 0, st>>>(g);
    else if (cls == 4) k_gram_f32<2, 0><<<grid, kThreads, 0, st>>>(g);
    else if (cls == 5) k_gram_f32<2, 1><<<grid, kThreads, 0, st>>>(g);
    else               k_gram_f32<2, 2><<<grid, kThreads, 0, st>>>(g);
    return hipGetLastError();
}

hipError_t launch_gram_f32(const GramPlan& p, const float* A, const float* G, int B, int T, int d_in, int d_out,
                           bool accumulate, float* sqnorm, float* partial, hipStream_t st, const ClipOut* co) {
    hipError_t e;
    if (T <= 32) {              // one tile pair per example (p.npairs == 1): the four waves split the contraction
        GramArgsF a;
        a.A = A; a.G = G; a.partial = partial;
        a.T = T; a.d_in = d_in; a.d_out = d_out;
        if (((d_in | d_out) & 3) == 0) k_gram_f32_small<true><<<(unsigned)B, kThreads, 0, st>>>(a);
        else                           k_gram_f32_small<false><<<(unsigned)B, kThreads, 0, st>>>(a);
        e = hipGetLastError();
    } else {
        const JointShape sh{T, d_in, d_out};
        const JointOperands op{reinterpret_cast<const uint16_t*>(A), reinterpret_cast<const uint16_t*>(G), nullptr, nullptr, 0};
        e = launch_gram_f32_layers(&sh, &op, &partial, 1, B, st);
    }
    if (e != hipSuccess) return e;
    return launch_finalize_partials(partial, B, p.npairs, accumulate, sqnorm, st, co);
}

}  // namespace dpk
