// The matrix-adaptation ES generation (CMA-ES of Table II in the form of
// Beyer and Sendhoff, 2017) apart from its two matrix products and the
// fitness pass: deviates, parent selection, recombination of the center and
// the path together with the factors of the rank-mu update, and the step
// size.  With s' the new path and d_i = M z_i the steps of the parents,
//     M [I + c_1/2 (s' s'^T - I) + c_w/2 (sum_i w_i z_i z_i^T - I)]
//   = (1 - (c_1 + c_w)/2) M + (M s') (c_1/2 s')^T + sum_i d_i (c_w/2 w_i z_i)^T,
// and M s' = (1 - c_s) M s + sqrt(mu_eff c_s (2 - c_s)) sum_i w_i d_i, so the
// update is one rank-(mu + 1) product of two factors that this file writes
// k-major ([term][column], so that a wave's operand loads are coalesced) and
// then applies to M in one streaming pass, and M s comes from the sampling
// product (the path rides along as an extra deviate row).
#include "evox_launch.hpp"

namespace evox {

namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));

// ---------------------------------------------------------------------------
// The sampling product Dm = Z M^T on the bf16 matrix cores, in fp32 precision.
// Each operand is the exact sum of three bf16 numbers, x = h + m + l (each the
// rounding of what the ones before leave: 8 + 8 + 8 bits), and of the nine
// products of pieces the six down to 2^-18 are summed in fp32; the three left
// out are below 2^-25 of the term, less than the rounding of one fp32 product.
// Six bf16 products cost 6 / 16 of one fp32 product on gfx950 (2.5 PFLOP/s
// against 157 TFLOP/s).
//
// That holds for 0 and for magnitudes of 2^-80 .. 2^56 in M and 2^-40 .. 2^56 in
// the path s (a deviate is 0 or within 2^-40 .. 2^3): the pieces are normal
// numbers, no product of them falls more than 2^-18 below 2^-120, and no sum of
// products overflows (2^56 2^56 of 2^15 columns), which the pieces of either sign
// would turn into a NaN.  A block that meets another element computes its tile
// again with fp32 products (v_mfma_f32_16x16x4f32), so that infinities and tiny
// numbers come out as they would without the split; a NaN stays one in either
// product.
//
// Z is split where it is drawn, into tiles of 3 pieces x 4 groups of 8 columns x
// zr rows that a block copies to LDS as they are (16 lanes of one column group
// read 256 consecutive bytes); M is read from memory straight into
// the operand registers -- lane l holds 8 consecutive k of row l % 16, a whole
// 128-byte line per row -- and split there, so it passes through no LDS and is
// split once per row tile.  Block: zr rows x 128 columns, 4 waves of zr x 32 (for
// zr = 112 7 x 2 tiles of v_mfma_f32_16x16x32_bf16, 84 per 32 columns of K).  zr is
// 112, or 32 or 64 where they hold every row, or 64 for two tiles of 113 .. 128
// rows: with 112 alone 16 samples padded sevenfold and populations of that kind
// lost up to 9 % to the fp32 product; a generation now takes, before and now, 201
// and 173 us (16 x 8192), 742 and 627 (30 x 16384), 317 and 287 (120 x 8192).
//
// At 101 x 16384 x 16384: 380 us (the fp32 matrix-core product of before took 560
// in k_gemm_nt16 and its split-K reduction), against 167 us for one pass over M at
// the copy rate, 148 us of matrix-core cycles at 2.4 GHz and 306 us at the rate a
// large bf16 library product reaches here; what is left is M's latency with two
// waves per SIMD.  A generation: 1002 -> 789 us; 4096 x 1830: 553 -> 487; 700 x
// 6000: 1156 -> 827; 50 x 500: 52 -> 48.  Pieces stored row by row ([112][32])
// cost 22M bank conflicts and 12 us; operand arrays of HIP's class vectors went to
// scratch (660 us); a loop exit between the steps of a group made every load of
// M wait at once (+11 us).
// Error against 64 bits, relative rms over the steps, before and now: D = 100
// 1.8e-7, 1.4e-7; 500 4.0e-7, 1.4e-7; 4096 3.4e-7, 2.5e-7; 8192 6.6e-7, 5.1e-7
// (one fp32 rounding per 32 columns and product of pieces, not per column pair);
// below D = 3, where one product's own rounding shows, the fp32 path is taken.
// ---------------------------------------------------------------------------
constexpr int kSpCols = 128;
constexpr uint32_t kSplitLo = (127 - 80) << 23, kPathLo = (127 - 40) << 23, kSplitHi = (127 + 56) << 23;

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// The two numbers rounded to bf16, packed.
__device__ __forceinline__ uint32_t pack_bf16(float a, float b)
{
    const bf16x2 t = __builtin_convertvector((f32x2){a, b}, bf16x2);
    return __builtin_bit_cast(uint32_t, t);
}

// The three pieces of a pair of numbers, packed.
__device__ __forceinline__ void split2(float a, float b, uint32_t &h, uint32_t &m, uint32_t &l)
{
    h = pack_bf16(a, b);
    const float a1 = a - __uint_as_float(h << 16), b1 = b - __uint_as_float(h & 0xffff0000u);
    m = pack_bf16(a1, b1);
    l = pack_bf16(a1 - __uint_as_float(m << 16), b1 - __uint_as_float(m & 0xffff0000u));
}

// Whether an element of the path cannot be split: not 0 and outside [2^-40, 2^56).
__device__ __forceinline__ bool odd_number(float x)
{
    const uint32_t e = __float_as_uint(x) & 0x7fffffffu;
    return e != 0 && (e < kPathLo || e >= kSplitHi);
}

// Deviates z_k (rows k < N, Philox stream 9 with the generation in the
// counter) and the path s (row N); columns D..ldx-1 zero.  Also their pieces.
__global__ __launch_bounds__(256) void k_mae_sample(MaeArgs a)
{
    const int64_t q4 = a.ldx / 4, total = (a.N + 1) * q4, kb = (a.D + 31) / 32;
    for (int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x; q < total; q += (int64_t)gridDim.x * 256) {
        const int64_t row = q / q4, c = q % q4;
        float4 v;
        if (row < a.N) {
            const float4 z = normal4((uint32_t)c, (uint32_t)row, a.t, STREAM_MAES, a.k0, a.k1);
            v.x = 4 * c + 0 < a.D ? z.x : 0.0f;
            v.y = 4 * c + 1 < a.D ? z.y : 0.0f;
            v.z = 4 * c + 2 < a.D ? z.z : 0.0f;
            v.w = 4 * c + 3 < a.D ? z.w : 0.0f;
        } else {
            v = *reinterpret_cast<const float4 *>(a.s + 4 * c);
            v.x = 4 * c + 0 < a.D ? v.x : 0.0f;
            v.y = 4 * c + 1 < a.D ? v.y : 0.0f;
            v.z = 4 * c + 2 < a.D ? v.z : 0.0f;
            v.w = 4 * c + 3 < a.D ? v.w : 0.0f;
        }
        *reinterpret_cast<float4 *>(a.Z + row * a.ldx + 4 * c) = v;
        if (4 * c >= 32 * kb) continue;  // padding past the last tile
        uint32_t p[3][2];
        split2(v.x, v.y, p[0][0], p[1][0], p[2][0]);
        split2(v.z, v.w, p[0][1], p[1][1], p[2][1]);
        const uint32_t rt = (uint32_t)row / (uint32_t)a.zr, rr = (uint32_t)row - rt * (uint32_t)a.zr;
        uint16_t *dst = a.Zs + (rt * kb + c / 8) * (96 * a.zr) + ((c % 8) / 2 * a.zr + rr) * 8 + 4 * (c % 2);
#pragma unroll
        for (int u = 0; u < 3; ++u)
            *reinterpret_cast<uint2 *>(dst + u * a.zr * 32) = make_uint2(p[u][0], p[u][1]);
    }
}

// K in steps of 32; the steps [s0, s1) of split z = blockIdx.x % splits.  With
// several splits the partial tile goes to work[z]; k_splitk_reduce adds them in
// order.  Operands in flight: M's next kSpDepth steps in registers, Z's next
// tile in registers and the one after that in the other LDS buffer.
constexpr int kSpDepth = 3;

template <int RB>  // blocks of 16 rows per tile
__global__ __launch_bounds__(256, 2) void k_mae_product(MaeArgs a, const float *M, int splits, float *work)
{
    constexpr int kSpRows = 16 * RB, kSpTile = 96 * kSpRows;  // rows, bf16 numbers of a tile of Z
    __shared__ __align__(16) uint16_t As[2][kSpTile];
    __shared__ int32_t odd;
    constexpr int NA = kSpTile / 8, QA = (NA + 255) / 256;  // 16-byte pieces of a tile, per thread
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, r16 = lane & 15, kg = lane >> 4;
    const int z = blockIdx.x % splits;
    const int64_t tn = (a.D + kSpCols - 1) / kSpCols, tile = blockIdx.x / splits;
    const int64_t rt = tile / tn, j0 = tile % tn * kSpCols + 32 * wave;
    const int steps = (int)((a.D + 31) / 32), per = (steps + splits - 1) / splits;
    const int s0 = z * per, s1 = s0 + per < steps ? s0 + per : steps;
    const int64_t rows = a.N + 1, i0 = rt * kSpRows;
    const u32x4 *At = reinterpret_cast<const u32x4 *>(a.Zs) + rt * steps * NA;

    // the lane's two rows of M (past the last row the last one, for columns that
    // are not stored; k past the last column is read from inside and zeroed)
    const float *mrow[2];
    bool in[2];
#pragma unroll
    for (int n = 0; n < 2; ++n) {
        const int64_t j = j0 + 16 * n + r16;
        in[n] = j < a.D;
        mrow[n] = M + (in[n] ? j : a.D - 1) * a.ldx;
    }
    f32x4 bq[kSpDepth][2][2];
    auto load_b = [&](f32x4 (&b)[2][2], int s) {
        const int64_t k = 32 * (int64_t)s + 8 * kg;
#pragma unroll
        for (int n = 0; n < 2; ++n)
#pragma unroll
            for (int h = 0; h < 2; ++h)
                b[n][h] = *reinterpret_cast<const f32x4 *>(mrow[n] + (k + 4 * h < a.ldx ? k + 4 * h : 0));
    };
    u32x4 aq[QA];
    auto load_a = [&](int s) {
#pragma unroll
        for (int u = 0; u < QA; ++u) {
            const int e = tid + 256 * u;  // the last round's spare threads copy the last piece again
            aq[u] = At[(int64_t)s * NA + (e < NA ? e : NA - 1)];
        }
    };
    auto store_a = [&](int buf) {
#pragma unroll
        for (int u = 0; u < QA; ++u) {
            const int e = tid + 256 * u;
            reinterpret_cast<u32x4 *>(As[buf])[e < NA ? e : NA - 1] = aq[u];
        }
    };
    auto lds_barrier = [] {  // fences LDS only: loads stay in flight
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
    };
    f32x4 acc[RB][2];
#pragma unroll
    for (int m = 0; m < RB; ++m)
#pragma unroll
        for (int n = 0; n < 2; ++n) acc[m][n] = (f32x4){0.f, 0.f, 0.f, 0.f};
    // the range of M's elements: greatest magnitude (NaN aside: it comes out of
    // either product), least bits of a magnitude other than 0, times 2, less 1
    float big = 0.0f;
    uint32_t small = 0xffffffffu;
    bool sodd = false;  // an element of the path in this slice cannot be split
    if (tid == 0) odd = a.D <= 2;

    if (s0 < s1) {
        const int last = s1 - 1;
        load_a(s0);
#pragma unroll
        for (int d = 0; d < kSpDepth; ++d) load_b(bq[d], s0 + d < last ? s0 + d : last);
        // behind the first loads, not before them
        if (rows - i0 <= kSpRows)
            for (int64_t k = 32 * (int64_t)s0 + tid; k < 32 * (int64_t)s1 && k < a.D; k += 256)
                sodd = sodd || odd_number(a.s[k]);
        store_a(0);
        load_a(s0 + 1 < last ? s0 + 1 : last);
        lds_barrier();
        for (int sb = s0; sb < s1; sb += kSpDepth) {
#pragma unroll
            for (int d = 0; d < kSpDepth; ++d) {
                // a last group's steps past s1 run on zeros: no branch leaves the
                // group, so every load is waited for by its own count
                const int s = sb + d, buf = (s - s0) & 1;
                store_a(buf ^ 1);
                load_a(s + 2 < last ? s + 2 : last);
                __builtin_amdgcn_sched_barrier(0);  // the loads keep this order, oldest needed first
                const int64_t k = 32 * (int64_t)s + 8 * kg;
                if (s >= s1 - 1) {  // the last step may pass the last column
#pragma unroll
                    for (int n = 0; n < 2; ++n)
#pragma unroll
                        for (int h = 0; h < 2; ++h)
#pragma unroll
                            for (int e = 0; e < 4; ++e)
                                bq[d][n][h][e] = s < s1 && k + 4 * h + e < a.D ? bq[d][n][h][e] : 0.0f;
                }
                // M's elements of this step: range, pieces
                uint32_t hp[2][4], mp[2][4], lp[2][4];
#pragma unroll
                for (int n = 0; n < 2; ++n)
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        const f32x4 v = bq[d][n][h];
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            big = fmaxf(big, fabsf(v[e]));
                            const uint32_t t = (__float_as_uint(v[e]) << 1) - 1u;  // 0: the greatest
                            small = t < small ? t : small;
                        }
                        split2(v[0], v[1], hp[n][2 * h], mp[n][2 * h], lp[n][2 * h]);
                        split2(v[2], v[3], hp[n][2 * h + 1], mp[n][2 * h + 1], lp[n][2 * h + 1]);
                    }
                load_b(bq[d], s + kSpDepth < last ? s + kSpDepth : last);
                __builtin_amdgcn_sched_barrier(0);
                bf16x8 bh[2], bm[2], bl[2];
#pragma unroll
                for (int n = 0; n < 2; ++n) {
                    bh[n] = __builtin_bit_cast(bf16x8, (u32x4){hp[n][0], hp[n][1], hp[n][2], hp[n][3]});
                    bm[n] = __builtin_bit_cast(bf16x8, (u32x4){mp[n][0], mp[n][1], mp[n][2], mp[n][3]});
                    bl[n] = __builtin_bit_cast(bf16x8, (u32x4){lp[n][0], lp[n][1], lp[n][2], lp[n][3]});
                }
                const uint16_t *src = As[buf] + (kg * kSpRows + r16) * 8;
#pragma unroll
                for (int m = 0; m < RB; ++m) {
                    const bf16x8 ah = *reinterpret_cast<const bf16x8 *>(src + m * 16 * 8);
                    const bf16x8 am = *reinterpret_cast<const bf16x8 *>(src + kSpRows * 32 + m * 16 * 8);
                    const bf16x8 al = *reinterpret_cast<const bf16x8 *>(src + 2 * kSpRows * 32 + m * 16 * 8);
                    // small terms first
#define EVOX_TERM(X, Y)                                                                                      \
    _Pragma("unroll") for (int n = 0; n < 2; ++n) acc[m][n] =                                                \
        __builtin_amdgcn_mfma_f32_16x16x32_bf16(X, Y[n], acc[m][n], 0, 0, 0)
                    EVOX_TERM(al, bh);
                    EVOX_TERM(ah, bl);
                    EVOX_TERM(am, bm);
                    EVOX_TERM(am, bh);
                    EVOX_TERM(ah, bm);
                    EVOX_TERM(ah, bh);
#undef EVOX_TERM
                }
                lds_barrier();
            }
        }
    }
    // the loop's barriers order this after the first value; every writer stores 1
    if (sodd || big >= __uint_as_float(kSplitHi) || small < 2u * kSplitLo - 1u) odd = 1;
    __syncthreads();
    if (odd) {
        // fp32 products: lane l holds k 4 u + kg of row r16, u = 0 .. 7
#pragma unroll
        for (int m = 0; m < RB; ++m)
#pragma unroll
            for (int n = 0; n < 2; ++n) acc[m][n] = (f32x4){0.f, 0.f, 0.f, 0.f};
        for (int s = s0; s < s1; ++s)
            for (int u = 0; u < 8; ++u) {
                const int64_t k = 32 * (int64_t)s + 4 * u + kg;
                float bv[2];
#pragma unroll
                for (int n = 0; n < 2; ++n) bv[n] = in[n] && k < a.D ? mrow[n][k] : 0.0f;
#pragma unroll
                for (int m = 0; m < RB; ++m) {
                    const int64_t i = i0 + 16 * m + r16;
                    const float av = i < rows && k < a.D ? a.Z[i * a.ldx + k] : 0.0f;
#pragma unroll
                    for (int n = 0; n < 2; ++n)
                        acc[m][n] = __builtin_amdgcn_mfma_f32_16x16x4f32(av, bv[n], acc[m][n], 0, 0, 0);
                }
            }
    }
    // result v of tile (m, n): row 16 m + 4 kg + v, column 16 n + r16
#pragma unroll
    for (int m = 0; m < RB; ++m)
#pragma unroll
        for (int n = 0; n < 2; ++n)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int64_t i = i0 + 16 * m + 4 * kg + v, j = j0 + 16 * n + r16;
                if (i < rows && j < a.D) {
                    if (splits > 1)
                        work[((int64_t)z * rows + i) * a.D + j] = acc[m][n][v];
                    else
                        a.Dm[i * a.ldx + j] = acc[m][n][v];
                }
            }
}

// sel[r] = the sample of rank r, for the mu best.
__global__ __launch_bounds__(256) void k_mae_select(MaeArgs a)
{
    const int64_t k = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (k >= a.N) return;
    const uint32_t r = a.rank[k];
    if (r < (uint32_t)a.mu) a.sel[r] = (int32_t)k;
}

// Factor terms r < mu, one thread per (column j, term r): At[r][j] = d_{r:N, j}
// and Bt[r][j] = c_w/2 w_r z_{r:N, j} (rounded once).
__global__ __launch_bounds__(256) void k_mae_gather(MaeArgs a)
{
    const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x, r = blockIdx.y;
    if (j >= a.D) return;
    const int64_t k = a.sel[r];
    a.At[r * a.ldf + j] = a.Dm[k * a.ldx + j];
    a.Bt[r * a.ldf + j] = (float)(a.hcw * a.w[r] * (double)a.Z[k * a.ldx + j]);
}

// Weighted parent sums over chunk c of kMaeChunk parents, one thread per
// column: wpart[c][0][j] = sum w_r z_{r:N, j}, wpart[c][1][j] = sum w_r d_{r:N, j}
// (fp64, parents in rank order).
__global__ __launch_bounds__(256) void k_mae_wsum(MaeArgs a)
{
    const int64_t j = (int64_t)blockIdx.x * 256 + threadIdx.x, c = blockIdx.y;
    if (j >= a.D) return;
    const int64_t r0 = c * kMaeChunk, r1 = r0 + kMaeChunk < a.mu ? r0 + kMaeChunk : a.mu;
    double zw = 0.0, dw = 0.0;
    // unrolled so that several parents' loads are in flight (same order)
#pragma unroll 8
    for (int64_t r = r0; r < r1; ++r) {
        const int64_t k = a.sel[r];
        const double wr = a.w[r];
        zw += wr * (double)a.Z[k * a.ldx + j];
        dw += wr * (double)a.Dm[k * a.ldx + j];
    }
    a.wpart[(2 * c) * a.D + j] = zw;
    a.wpart[(2 * c + 1) * a.D + j] = dw;
}

// One thread per column j: <z>_w and <d>_w from the chunk sums (in chunk
// order), y_j <- y_j + sigma <d>_w, s_j <- (1 - c_s) s_j + c_z <z>_w, the last
// factor term (At[mu][j] = (M s')_j, Bt[mu][j] = c_1/2 s'_j; the terms past mu
// and the columns past D are zero from creation), and the block's sum of
// s'_j^2 (fp64, fixed order).  Term r < mu of the factors is
//     At[r][j] = d_{r:N, j},  Bt[r][j] = c_w/2 w_r z_{r:N, j}  (k_mae_gather).
__global__ __launch_bounds__(kMaeBlock) void k_mae_recombine(MaeArgs a, int64_t nchunks)
{
    __shared__ double red[kMaeBlock];
    const int64_t j = (int64_t)blockIdx.x * kMaeBlock + threadIdx.x;
    double sq = 0.0;
    if (j < a.D) {
        double zw = 0.0, dw = 0.0;
#pragma unroll 8
        for (int64_t c = 0; c < nchunks; ++c) {
            zw += a.wpart[(2 * c) * a.D + j];
            dw += a.wpart[(2 * c + 1) * a.D + j];
        }
        const double sig = (double)*a.sigma, keep = 1.0 - a.cs;
        const float sn = (float)(keep * (double)a.s[j] + a.cz * zw);
        a.At[a.mu * a.ldf + j] = (float)(keep * (double)a.Dm[a.N * a.ldx + j] + a.cz * dw);
        a.Bt[a.mu * a.ldf + j] = (float)(a.hc1 * (double)sn);
        a.y[j] = (float)((double)a.y[j] + sig * dw);
        a.s[j] = sn;
        sq = (double)sn * (double)sn;
    }
    red[threadIdx.x] = sq;
    __syncthreads();
    for (int w = kMaeBlock / 2; w > 0; w /= 2) {
        if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) a.part[blockIdx.x] = red[0];
}

// sigma <- sigma exp(c_s/d_s (|s'| / chi_D - 1)), |s'|^2 from the block sums
// in a fixed order.
__global__ __launch_bounds__(256) void k_mae_sigma(MaeArgs a, int64_t nparts)
{
    __shared__ double red[256];
    double acc = 0.0;
    for (int64_t q = threadIdx.x; q < nparts; q += 256) acc += a.part[q];
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int w = 128; w > 0; w /= 2) {
        if (threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) *a.sigma = (float)((double)*a.sigma * exp(a.damp * (sqrt(red[0]) / a.chi - 1.0)));
}

// M <- beta M + At^T Bt over 2 STEPS factor terms (the factors hold zeros
// past the mu + 1 real terms and past column D, up to their padded extents:
// kp = 2 STEPS terms, a pitch ldf that is a multiple of 128, so no operand
// load needs a guard).  A block of four waves owns a 128 x 64 tile of M, each
// wave a 32 x 64 slice of it accumulated in two 32x32x2 MFMA tiles.  The
// block first issues its operand loads (the 128 rows of At and 64 columns
// of Bt over all terms, float4 from the k-major factors), then each wave
// issues the 32 loads of its slice of M; the operands go to LDS as soon as
// they arrive (loads complete in order, so the slice is still on its way
// from HBM) and the products read them from LDS while the slice arrives.
// LDS holds each term pair interleaved ([pair][row][term of the pair]) so
// that lane l = col + 32 h reads float 2 col + h of a pair: 64 consecutive
// floats, no bank conflicts.  The barrier fences LDS only, keeping the
// slice's loads in flight.  Rows past D read as zero and are not stored.
// Waves per SIMD the staged operands leave room for: four blocks of up to
// 40 KB of LDS per CU, three past that.
template <int STEPS>
constexpr int kMaeRankWaves = STEPS * 48 * 32 <= 160 * 1024 / 4 ? 4 : 3;

template <int STEPS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(kMaeRankWaves<STEPS>))) void k_mae_rank(MaeArgs a, float *M,
                                                                                           float beta)
{
    constexpr int NA = STEPS * 32, NI = STEPS * 48, PER = (NI + 255) / 256;  // float4 pairs of terms to stage
    __shared__ float4 sA[STEPS * 64], sB[STEPS * 32];
    const int tid = threadIdx.x, lane = tid % 64, col = lane % 32, h = lane / 32, w = tid / 64;
    const int64_t tn = (a.D + 63) / 64, ldf = a.ldf, ld = a.ldx;
    const int64_t I0 = ((int64_t)blockIdx.x / tn) * 128, j0 = ((int64_t)blockIdx.x % tn) * 64;
    const int64_t i0 = I0 + 32 * w;
    float4 lo[PER], hi[PER];
#pragma unroll
    for (int p = 0; p < PER; ++p) {
        // the last round's spare threads load the last item again (no
        // branch around the loads, which would wait for them)
        const int it = tid + 256 * p < NI ? tid + 256 * p : NI - 1;
        const bool isA = it < NA;
        const int s = isA ? it / 32 : (it - NA) / 16, q = isA ? it % 32 : (it - NA) % 16;
        const float *f = (isA ? a.At + I0 : a.Bt + j0) + 2 * s * ldf + 4 * q;
        lo[p] = *reinterpret_cast<const float4 *>(f);
        hi[p] = *reinterpret_cast<const float4 *>(f + ldf);
    }
    // The wave's slice of M through a buffer descriptor based at its first
    // element and ending at the end of M: rows past D fall outside its range
    // and read as zero (they are not stored).  The row offset sits in the
    // lane offset because the range check ignores the scalar offset.  M is
    // read and written once per pass, with the non-temporal policy (aux 2),
    // which keeps the staged factors in the L2.
    const int64_t wi0 = I0 + 32 * __builtin_amdgcn_readfirstlane(w);  // = i0, known to be wave-uniform
    const int64_t left = wi0 < a.D ? ((a.D - wi0) * ld - j0) * 4 : 0;  // bytes from the slice to the end of M
    const __amdgpu_buffer_rsrc_t mr = __builtin_amdgcn_make_buffer_rsrc(
        M + (wi0 < a.D ? wi0 * ld + j0 : 0), 0, (int)(left < 0x7fffffffLL ? left : 0x7fffffffLL), 0x00020000);
    float old[2][16];
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const int off = (((v / 4) * 8 + h * 4 + v % 4) * (int)ld + col) * 4;
        old[0][v] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(mr, off, 0, 2));  // the load returns bits
        old[1][v] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(mr, off + 128, 0, 2));
    }
#pragma unroll
    for (int p = 0; p < PER; ++p) {
        const int it = tid + 256 * p;
        if (p + 1 < PER || it < NI) {
            const bool isA = it < NA;
            const int s = isA ? it / 32 : (it - NA) / 16, q = isA ? it % 32 : (it - NA) % 16;
            float4 *d = isA ? sA + s * 64 + 2 * q : sB + s * 32 + 2 * q;
            d[0] = make_float4(lo[p].x, hi[p].x, lo[p].y, hi[p].y);
            d[1] = make_float4(lo[p].z, hi[p].z, lo[p].w, hi[p].w);
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
    if (i0 >= a.D) return;
    const float *la = reinterpret_cast<const float *>(sA) + (32 * w + col) * 2 + h;
    const float *lb = reinterpret_cast<const float *>(sB) + col * 2 + h;
    f32x16 acc[2];
#pragma unroll
    for (int n = 0; n < 2; ++n)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[n][v] = 0.0f;
#pragma unroll
    for (int s = 0; s < STEPS; ++s) {
        const float av = la[s * 256], b0 = lb[s * 128], b1 = lb[s * 128 + 64];
        acc[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(av, b0, acc[0], 0, 0, 0);
        acc[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(av, b1, acc[1], 0, 0, 0);
    }
    if (j0 + 64 <= a.D) {
        // every column is inside the matrix: store through the descriptor,
        // which drops the rows past D
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int off = (((v / 4) * 8 + h * 4 + v % 4) * (int)ld + col) * 4;
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(fmaf(1.0f, acc[0][v], beta * old[0][v])), mr, off, 0, 2);
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(fmaf(1.0f, acc[1][v], beta * old[1][v])), mr, off + 128,
                                                  0, 2);
        }
        return;
    }
#pragma unroll
    for (int n = 0; n < 2; ++n)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int64_t i = i0 + (v / 4) * 8 + h * 4 + v % 4, j = j0 + 32 * n + col;
            if (i < a.D && j < a.D) M[i * ld + j] = fmaf(1.0f, acc[n][v], beta * old[n][v]);
        }
}

// The same update for any number of terms (a.kp, a multiple of 32): each
// wave owns a 32 x 64 tile of M and loads its MFMA operands directly from the
// k-major factors (lane l: row or column l % 32 of term 2 step + l / 32, one
// 128-byte line per half wave), 16 steps at a time, double-buffered: the
// next block's loads are in flight while the current block's products run.
// The tile of M is loaded first.  It holds two blocks of operands at one
// wave per SIMD, which measured faster than 2 or 3 waves with 8-step blocks.
__global__ __launch_bounds__(256) void k_mae_rank_any(MaeArgs a, float *M, float beta)
{
    constexpr int CH = 16;
    const int lane = threadIdx.x % 64, col = lane % 32, h = lane / 32;
    const int64_t tn = (a.D + 63) / 64;
    const int64_t wave = (int64_t)blockIdx.x * 4 + threadIdx.x / 64;
    const int64_t i0 = (wave / tn) * 32, j0 = (wave % tn) * 64;
    if (i0 >= a.D) return;
    float old[2][16];
#pragma unroll
    for (int n = 0; n < 2; ++n)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int64_t i = i0 + (v / 4) * 8 + h * 4 + v % 4, j = j0 + 32 * n + col;
            old[n][v] = (i < a.D && j < a.D) ? M[i * a.ldx + j] : 0.0f;
        }
    f32x16 acc[2];
#pragma unroll
    for (int n = 0; n < 2; ++n)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[n][v] = 0.0f;
    const float *pa = a.At + h * a.ldf + i0 + col;
    const float *pb = a.Bt + h * a.ldf + j0 + col;
    float av[2][CH], b0[2][CH], b1[2][CH];
    auto load = [&](int buf, int64_t c0) {
#pragma unroll
        for (int t = 0; t < CH; ++t) {
            const int64_t off = 2 * (c0 + t) * a.ldf;
            av[buf][t] = pa[off];
            b0[buf][t] = pb[off];
            b1[buf][t] = pb[off + 32];
        }
    };
    auto products = [&](int buf) {
#pragma unroll
        for (int t = 0; t < CH; ++t) {
            acc[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[buf][t], b0[buf][t], acc[0], 0, 0, 0);
            acc[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[buf][t], b1[buf][t], acc[1], 0, 0, 0);
        }
    };
    const int64_t steps = a.kp / 2;
    load(0, 0);
    for (int64_t c0 = 0; c0 < steps; c0 += 2 * CH) {
        if (c0 + CH < steps) load(1, c0 + CH);
        products(0);
        if (c0 + CH < steps) {
            if (c0 + 2 * CH < steps) load(0, c0 + 2 * CH);
            products(1);
        }
    }
#pragma unroll
    for (int n = 0; n < 2; ++n)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int64_t i = i0 + (v / 4) * 8 + h * 4 + v % 4, j = j0 + 32 * n + col;
            if (i < a.D && j < a.D) M[i * a.ldx + j] = fmaf(1.0f, acc[n][v], beta * old[n][v]);
        }
}

__global__ __launch_bounds__(256) void k_mae_identity(float *M, int64_t D, int64_t ldx)
{
    const int64_t total = D * ldx;
    for (int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x; q < total; q += (int64_t)gridDim.x * 256)
        M[q] = (q / ldx == q % ldx) ? 1.0f : 0.0f;
}

unsigned blocks_for(int64_t n, int64_t per, int64_t cap)
{
    const int64_t b = (n + per - 1) / per;
    return (unsigned)(b < 1 ? 1 : b > cap ? cap : b);
}

}  // namespace

hipError_t launch_mae_sample(const MaeArgs &a, hipStream_t s)
{
    hipLaunchKernelGGL(k_mae_sample, dim3(blocks_for((a.N + 1) * (a.ldx / 4), 256, 16384)), dim3(256), 0, s, a);
    return hipGetLastError();
}

int occupancy_mae_product(int64_t zr)
{
    const auto k = zr == 32 ? k_mae_product<2> : zr == 64 ? k_mae_product<4> : k_mae_product<7>;
    int n = 0;
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k, 256, 0) == hipSuccess ? n : 0;
}

hipError_t launch_mae_product(const MaeArgs &a, const float *M, int splits, float *work, hipStream_t s)
{
    if (splits < 1 || (splits > 1 && !work)) return hipErrorInvalidValue;
    const int64_t tiles = ((a.D + kSpCols - 1) / kSpCols) * ((a.N + a.zr) / a.zr);
    const auto k = a.zr == 32 ? k_mae_product<2> : a.zr == 64 ? k_mae_product<4> : k_mae_product<7>;
    hipLaunchKernelGGL(k, dim3((unsigned)(tiles * splits)), dim3(256), 0, s, a, M, splits, work);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess || splits == 1) return e;
    return launch_splitk_reduce(GemmArgs{a.N + 1, a.D, a.D, 1.0f, nullptr, 0, nullptr, 0, 0.0f, a.Dm, a.ldx}, splits,
                                work, s);
}

hipError_t launch_mae_select(const MaeArgs &a, hipStream_t s)
{
    hipLaunchKernelGGL(k_mae_select, dim3(blocks_for(a.N, 256, 1 << 20)), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_mae_recombine(const MaeArgs &a, hipStream_t s)
{
    const int64_t nparts = (a.D + kMaeBlock - 1) / kMaeBlock, cols = (a.D + 255) / 256;
    const int64_t nchunks = (a.mu + kMaeChunk - 1) / kMaeChunk;
    hipLaunchKernelGGL(k_mae_gather, dim3((unsigned)cols, (unsigned)a.mu), dim3(256), 0, s, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_mae_wsum, dim3((unsigned)cols, (unsigned)nchunks), dim3(256), 0, s, a);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(k_mae_recombine, dim3((unsigned)nparts), dim3(kMaeBlock), 0, s, a, nchunks);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(k_mae_sigma, dim3(1), dim3(256), 0, s, a, nparts);
    return hipGetLastError();
}

hipError_t launch_mae_rank(const MaeArgs &a, float *M, float beta, hipStream_t s)
{
    const int64_t waves = ((a.D + 31) / 32) * ((a.D + 63) / 64);
    const dim3 grid_any((unsigned)((waves + 3) / 4)), block(256);
    const dim3 grid((unsigned)(((a.D + 127) / 128) * ((a.D + 63) / 64)));
    const int64_t steps = (a.mu + 2) / 2;  // ceil((mu + 1) / 2)
    if (a.ldf % 128 != 0 || (steps <= kMaeRankUnrolled && a.kp != 2 * steps)) return hipErrorInvalidValue;
    switch (steps > kMaeRankUnrolled ? 0 : steps) {
#define EVOX_RANK_CASE(S) \
    case S: hipLaunchKernelGGL((k_mae_rank<S>), grid, block, 0, s, a, M, beta); break;
        EVOX_RANK_CASE(1) EVOX_RANK_CASE(2) EVOX_RANK_CASE(3) EVOX_RANK_CASE(4) EVOX_RANK_CASE(5)
        EVOX_RANK_CASE(6) EVOX_RANK_CASE(7) EVOX_RANK_CASE(8) EVOX_RANK_CASE(9) EVOX_RANK_CASE(10)
        EVOX_RANK_CASE(11) EVOX_RANK_CASE(12) EVOX_RANK_CASE(13) EVOX_RANK_CASE(14) EVOX_RANK_CASE(15)
        EVOX_RANK_CASE(16) EVOX_RANK_CASE(17) EVOX_RANK_CASE(18) EVOX_RANK_CASE(19) EVOX_RANK_CASE(20)
        EVOX_RANK_CASE(21) EVOX_RANK_CASE(22) EVOX_RANK_CASE(23) EVOX_RANK_CASE(24) EVOX_RANK_CASE(25)
        EVOX_RANK_CASE(26) EVOX_RANK_CASE(27) EVOX_RANK_CASE(28) EVOX_RANK_CASE(29) EVOX_RANK_CASE(30)
        EVOX_RANK_CASE(31) EVOX_RANK_CASE(32)
#undef EVOX_RANK_CASE
        default: hipLaunchKernelGGL(k_mae_rank_any, grid_any, block, 0, s, a, M, beta); break;
    }
    return hipGetLastError();
}

hipError_t launch_mae_identity(float *M, int64_t D, int64_t ldx, hipStream_t s)
{
    hipLaunchKernelGGL(k_mae_identity, dim3(blocks_for(D * ldx, 256, 16384)), dim3(256), 0, s, M, D, ldx);
    return hipGetLastError();
}

}  // namespace evox
