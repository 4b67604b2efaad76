// NSGA-II on DTLZ1 (Table II; the multi-objective scaling experiment of
// Sec. VII-A-2, whose speed-up the paper attributes to computing the dominance
// relations in parallel).  Deb, Pratap, Agarwal, Meyarivan (2002):
//   variation   crowded binary tournaments, simulated binary crossover and
//               polynomial mutation (one thread per pair and variable, fp64);
//   objectives  DTLZ1 (one wave per row, fp64: its g is a difference of
//               numbers near 100 k that fp32 would not resolve near the front);
//   sorting     the points in a coarse order of the first objective, the
//               dominance of every pair that this order leaves open as one bit
//               (a row of bits per point: its dominators), then fronts one at
//               a time: the unassigned points with no unassigned dominator form
//               the next front, whose members are appended to a list (fronts
//               stored contiguously);
//   crowding    each front member's position in every objective's order of
//               (value, index) by counting within its front (tiles of the
//               front through LDS), then the distance summed objective by
//               objective in that order;
//   selection   whole fronts, then the last front's members of largest
//               crowding distance (lower index on ties) by counting, and a
//               compaction that keeps the merged order.
#include "evox_launch.hpp"

#include <cmath>
#include <type_traits>

namespace evox {

namespace {

// points per LDS tile of the kernels that compare within fronts: short, since a
// front's pairs are few and more tiles put more waves on them (16,384 x 100,
// tiles of 512 / 128: order 61 / 32 us, truncation 16 / 7)
constexpr int kSpan = 128;
constexpr double kPi = 3.14159265358979323846;

__device__ __forceinline__ int64_t crowded_winner(int64_t a, int64_t b, const int32_t *front, const double *crowd)
{
    if (front[a] != front[b]) return front[a] < front[b] ? a : b;
    if (crowd[a] != crowd[b]) return crowd[a] > crowd[b] ? a : b;
    return a < b ? a : b;
}

// Polynomial mutation of x in [0, 1] with draw u and index eta (the bounded
// form of Deb and Goyal): u < 1/2 lowers x by 1 - (2u + (1 - 2u)(1 - x)^(eta+1))
// ^(1/(eta+1)), u >= 1/2 raises it by 1 - (2(1 - u) + 2(u - 1/2) x^(eta+1))
// ^(1/(eta+1)); clipped to [0, 1].
// One pair of powers for either half, so that a wave with both runs them once.
__device__ double poly_mutate(double x, double u, double eta)
{
    const double e1 = eta + 1.0, inv = 1.0 / e1;
    const bool low = u < 0.5;
    const double q = pow(low ? 1.0 - x : x, e1);
    const double r = pow(low ? 2.0 * u + (1.0 - 2.0 * u) * q : 2.0 * (1.0 - u) + 2.0 * (u - 0.5) * q, inv);
    const double y = x + (low ? r - 1.0 : 1.0 - r);
    return y < 0.0 ? 0.0 : y > 1.0 ? 1.0 : y;
}

// Offspring rows 2p and 2p + 1, variable j (one thread each): parents from
// the tournaments (w of Philox(0, p, t, 10): candidates floor(w_q N / 2^32),
// (w_0, w_1) and (w_2, w_3)); crossover and mutation draws from Philox(j, p,
// t, 11) and (j, p, t, 12).
__global__ __launch_bounds__(256) void k_nsga_var(NsgaVarArgs a)
{
    const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x, H = a.N / 2;
    if (q >= H * a.D) return;
    const int64_t p = q / a.D, j = q % a.D;
    const U4 ws = philox(0u, (uint32_t)p, a.t, STREAM_NSGA_SEL, a.k0, a.k1);
    const uint64_t n = (uint64_t)a.N;
    const int64_t c0 = (int64_t)(((uint64_t)ws.x * n) >> 32), c1 = (int64_t)(((uint64_t)ws.y * n) >> 32);
    const int64_t c2 = (int64_t)(((uint64_t)ws.z * n) >> 32), c3 = (int64_t)(((uint64_t)ws.w * n) >> 32);
    const int64_t pa = crowded_winner(c0, c1, a.front, a.crowd), pb = crowded_winner(c2, c3, a.front, a.crowd);
    const U4 w = philox((uint32_t)j, (uint32_t)p, a.t, STREAM_NSGA_VAR, a.k0, a.k1);
    const U4 v = philox((uint32_t)j, (uint32_t)p, a.t, STREAM_NSGA_MUT, a.k0, a.k1);
    const double ec = a.eta_c, em = a.eta_m, pm = 1.0 / (double)a.D;
    const double u = (double)u01(w.x);
    const double ie = 1.0 / (ec + 1.0), ne = -1.0 / (ec + 1.0);
    double beta = pow(u <= 0.5 ? 2.0 * u : 2.0 - 2.0 * u, u <= 0.5 ? ie : ne);
    if (w.y & 1u) beta = -beta;
    if ((double)u01(w.y) >= 0.5) beta = 1.0;
    const double xa = (double)a.X[pa * a.ldx + j], xb = (double)a.X[pb * a.ldx + j];
    const double y[2] = {0.5 * (xa + xb) + 0.5 * beta * (xa - xb), 0.5 * (xa + xb) - 0.5 * beta * (xa - xb)};
    const uint32_t coin[2] = {w.z, w.w}, mu[2] = {v.x, v.y};
    float out[2];
    bool mut[2];
#pragma unroll
    for (int c = 0; c < 2; ++c) {
        out[c] = (float)(y[c] < 0.0 ? 0.0 : y[c] > 1.0 ? 1.0 : y[c]);
        mut[c] = (double)u01(coin[c]) < pm;
    }
    // one in D variables mutates, one child at a time: a wave passes through
    // the powers once unless both children of a lane mutate
    while (mut[0] | mut[1]) {
        const bool first = mut[0];
        const float m = (float)poly_mutate((double)(first ? out[0] : out[1]), (double)u01(first ? mu[0] : mu[1]), em);
        out[0] = first ? m : out[0];
        out[1] = first ? out[1] : m;
        mut[1] = first && mut[1];
        mut[0] = false;
    }
    a.Q[2 * p * a.ldx + j] = out[0];
    a.Q[(2 * p + 1) * a.ldx + j] = out[1];
}

// DTLZ1 of row r (one wave): g = 100 (k + sum_{i >= M-1} ((x_i - 1/2)^2 -
// cos(20 pi (x_i - 1/2)))), f_0 = (1 + g)/2 x_0 ... x_{M-2}, f_m = (1 + g)/2
// x_0 ... x_{M-2-m} (1 - x_{M-1-m}); fp64, each objective rounded once.
// Behind the nold rows of objectives Fold, which are copied.  hist (nullable):
// the counts of the coarse order, cleared for the sort that follows.
__global__ __launch_bounds__(256) void k_nsga_dtlz1(const float *X, int64_t n, int64_t D, int64_t ldx, int32_t M,
                                                    const float *Fold, int64_t nold, float *F, uint32_t *hist)
{
    const int64_t r = (int64_t)blockIdx.x * 4 + threadIdx.x / 64;
    const int lane = threadIdx.x % 64;
    if (hist && blockIdx.x == 0)
        for (int q = threadIdx.x; q <= kNsgaSplit; q += 256) hist[q] = 0;
    if (r >= n) {
        const int64_t q = (r - n) * 64 + lane;
        if (q < nold * M) F[q] = Fold[q];
        return;
    }
    const float *x = X + r * ldx;
    double acc = 0.0;
    for (int64_t i = M - 1 + lane; i < D; i += 64) {
        const double d = (double)x[i] - 0.5;
        acc += d * d - cos(20.0 * kPi * d);
    }
    for (int o = 32; o > 0; o /= 2) acc += __shfl_xor(acc, o);
    if (lane < M) {
        const int m = lane;
        const double g = 100.0 * ((double)(D - M + 1) + acc);
        double f = 0.5 * (1.0 + g);
        for (int i = 0; i < M - 1 - m; ++i) f *= (double)x[i];
        if (m > 0) f *= 1.0 - (double)x[M - 1 - m];
        F[(nold + r) * M + m] = (float)f;
    }
}

// Objectives of a point padded to P = 4 or 8 floats in LDS (read back as
// float4 broadcasts: every lane of a wave reads the same point).
template <int P>
__device__ __forceinline__ void load_pad(float *dst, const float *F, int64_t row, int32_t M)
{
#pragma unroll
    for (int m = 0; m < P; ++m) dst[m] = m < M ? F[row * M + m] : 0.0f;
}

// Dominance of b by a for M objectives known at compile time (comparisons as
// written: NaN neither dominates nor is dominated differently than in the
// definition).
template <int M>
__device__ __forceinline__ bool dominates_t(const float *a, const float *b)
{
    bool worse = false, better = false;
#pragma unroll
    for (int m = 0; m < M; ++m) {
        worse |= a[m] > b[m];
        better |= a[m] < b[m];
    }
    return !worse && better;
}

// ---------------------------------------------------------------------------
// Pairs.  The points are taken in a coarse order of the first objective
// (buckets between 1024 sampled splitters; positions 0 .. n - 1, ord[pos] the
// point), in chunks of kNsgaChunk positions.  A chunk whose least first
// objective is above a point's chunk's greatest holds no dominator of it, one
// whose greatest is below the other's least dominates it in the first objective
// strictly, so that the others decide alone: half of the pairs are never
// looked at and most of the rest take M - 1 comparisons instead of 2M.  The
// order need not be exact: chunks that overlap are compared in full.
//
// The dominators of a point are bits, four words (a group) per 128 positions,
// bit 31 - q of word w for position 32 w + q (a compare and an add-with-carry
// per pair).  W holds them by chunk of points, then group, then point, so that a
// wave stores a group of its 64 points as one kilobyte.  A front is
// then found without a count: a point waits on the first group of four words
// (ptr) in which it has an unassigned dominator, and only when that group
// clears are its later groups searched, so all the fronts together read each
// of them about once.
//
// 32768 points, 3 objectives: coarse order 33 us and bits 81, against 240
// for counting dominators over all pairs; fronts 12 us each, against 35 for
// marking the points whose count is zero and subtracting their dominance.
// ---------------------------------------------------------------------------
constexpr int kSplit = kNsgaSplit, kPlaceBits = 17;  // sampled splitters; bits of a place in a bucket

__device__ __forceinline__ uint32_t ordered(float v)
{
    const uint32_t b = __float_as_uint(v);
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

// One thread per point: its bucket of the first objective and its place among
// the bucket's points (any order), packed; every block sorts the samples for
// itself.  hist is zero before.
__global__ __launch_bounds__(1024) void k_nsga_assign(const float *F, int32_t n, int32_t M, uint32_t *hist,
                                                      uint32_t *place)
{
    __shared__ uint32_t split[kSplit];
    const int tid = threadIdx.x, i = blockIdx.x * 1024 + tid;
    split[tid] = ordered(F[(int64_t)tid * n / kSplit * M]);
    const uint32_t key = i < n ? ordered(F[(int64_t)i * M]) : 0u;
    for (int k = 2; k <= kSplit; k *= 2)  // bitonic sort
        for (int j = k / 2; j > 0; j /= 2) {
            __syncthreads();
            const uint32_t a = split[tid], b = split[tid ^ j];
            __syncthreads();
            split[tid] = ((tid & k) == 0) == ((tid & j) == 0) ? (a < b ? a : b) : (a < b ? b : a);
        }
    __syncthreads();
    uint32_t lo = 0;  // number of splitters below the key: 0 .. kSplit
#pragma unroll
    for (int w = kSplit / 2; w >= 1; w /= 2) lo += split[lo + w - 1] < key ? w : 0;
    lo += split[lo] < key ? 1 : 0;
    if (i < n) place[i] = lo << kPlaceBits | atomicAdd(hist + lo, 1u);
}

// ord: every block scans the buckets' counts and places its points.
__global__ __launch_bounds__(1024) void k_nsga_place(int32_t n, const uint32_t *hist, const uint32_t *place,
                                                     int32_t *ord)
{
    __shared__ uint32_t off[kSplit + 1], wsum[16];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, i = blockIdx.x * 1024 + tid;
    const uint32_t c = hist[tid], p = i < n ? place[i] : 0u;
    uint32_t inc = c;
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t o = __shfl_up(inc, d, 64);
        if (lane >= d) inc += o;
    }
    if (lane == 63) wsum[wave] = inc;
    __syncthreads();
    uint32_t base = 0;
    for (int w = 0; w < wave; ++w) base += wsum[w];
    off[tid] = base + inc - c;
    if (tid == 1023) off[kSplit] = base + inc;
    __syncthreads();
    if (i < n) ord[off[p >> kPlaceBits] + (p & ((1u << kPlaceBits) - 1u))] = i;
}

// One block per chunk: the objectives in that order, padded to P floats
// (positions past n hold +inf, which dominates nothing), the range of the
// chunk's first objective (all of the line where it holds a NaN), and the
// state of the front search: every point unassigned, waiting on nothing.
template <int M>
__global__ __launch_bounds__(kNsgaChunk) void k_nsga_gather(NsgaSortArgs a)
{
    constexpr int P = M <= 4 ? 4 : 8;
    __shared__ float lo[kNsgaChunk / 64], hi[kNsgaChunk / 64];
    const int64_t pos = (int64_t)blockIdx.x * kNsgaChunk + threadIdx.x;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    float v[P];
#pragma unroll
    for (int m = 0; m < P; ++m) v[m] = m < M ? INFINITY : 0.0f;
    float l = INFINITY, h = -INFINITY;
    if (pos < a.n) {
        const int32_t i = a.ord[pos];
#pragma unroll
        for (int m = 0; m < M; ++m) v[m] = a.F[(int64_t)i * M + m];
        l = v[0] == v[0] ? v[0] : -INFINITY;
        h = v[0] == v[0] ? v[0] : INFINITY;
        a.front[i] = -1;
        a.ptr[pos] = kNsgaNoWord;
#pragma unroll
        for (int m = 0; m < M; ++m) {
            a.pos[m * a.cap + pos] = 0;
            // every slot of the per-objective orders holds a valid index even
            // if the order kernel were handed values without a total order
            a.sorted[m * a.cap + pos] = 0;
        }
    }
#pragma unroll
    for (int q = 0; q < P / 4; ++q)
        reinterpret_cast<float4 *>(a.Fs)[pos * (P / 4) + q] =
            make_float4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
#pragma unroll
    for (int m = 0; m < nsga_rest(M); ++m) a.Fr[pos * nsga_rest(M) + m] = m + 1 < M ? v[m + 1 < M ? m + 1 : 0] : 0.0f;
    for (int d = 32; d >= 1; d /= 2) {
        l = fminf(l, __shfl_xor(l, d, 64));
        h = fmaxf(h, __shfl_xor(h, d, 64));
    }
    if (lane == 0) {
        lo[wave] = l;
        hi[wave] = h;
    }
    // the mask of unassigned points: two words of 32 positions per wave
    if (lane < 2) {
        const int64_t p0 = pos - lane + 32 * lane, left = a.n - p0;
        a.mask[p0 / 32] = left >= 32 ? 0xffffffffu : left <= 0 ? 0u : ~(0xffffffffu >> left);
    }
    if (blockIdx.x == 0 && threadIdx.x < kNsgaPeelBatch) a.len[threadIdx.x] = 0;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kNsgaChunk / 64; ++w) {
            l = fminf(l, lo[w]);
            h = fmaxf(h, hi[w]);
        }
        a.range[2 * blockIdx.x] = l;
        a.range[2 * blockIdx.x + 1] = h;
    }
}

// Group g of point p of chunk ic.
__device__ __forceinline__ int64_t w_index(int64_t chunks, int64_t ic, int64_t g, int p)
{
    return (ic * 2 * chunks + g) * kNsgaChunk + p;
}

// Whether chunk jc can hold dominators of chunk ic's points.
__device__ __forceinline__ bool chunk_open(const float *range, int64_t ic, int64_t jc)
{
    return range[2 * jc] <= range[2 * ic + 1];
}

// 2 acc + the lane's bit of a comparison's lane mask: one add with carry (the
// compiler makes two instructions of it).
__device__ __forceinline__ uint32_t shift_in(uint32_t acc, uint64_t mask)
{
    uint64_t carry;
    asm("v_addc_co_u32_e64 %0, %1, %0, %0, %2" : "+v"(acc), "=&s"(carry) : "s"(mask));
    return acc;
}

// Bits of one chunk of 256 positions jc against the point fi: 8 words.  The
// comparisons stay lane masks in scalar registers (dominates_t: no a > b, some
// a < b), so a strict pair is M - 1 vector compares and the add.
// The positions' objectives are the same in every lane and come through scalar
// loads, 64 bytes at a time: the strict pairs' from an array without the first
// objective (from the padded one a load per position: 145 us instead of 121 with four chunks
// per block).
template <int M, bool STRICT>
__device__ __forceinline__ void chunk_bits(const float *__restrict__ fs, int64_t jc, const float (&fi)[M],
                                           uint32_t (&out)[8])
{
    constexpr int P = STRICT ? nsga_rest(M) : M <= 4 ? 4 : 8, kUle = 13, kOlt = 4;  // predicates: not >, <
    constexpr int U = 64 / P < 32 ? 64 / P : 32;                                  // positions per batch
    const float *src = fs + jc * kNsgaChunk * P;
#pragma unroll
    for (int w = 0; w < 8; ++w) {
        uint32_t acc = 0;
#pragma unroll 1
        for (int q0 = 0; q0 < 32; q0 += U) {
            float v[U * P];
#pragma unroll
            for (int e = 0; e < U * P; ++e) v[e] = src[(32 * w + q0) * P + e];
#pragma unroll
            for (int q = 0; q < U; ++q) {
                uint64_t le = ~(uint64_t)0, lt = 0;
#pragma unroll
                for (int m = STRICT ? 1 : 0; m < M; ++m) {
                    const float vm = v[q * P + m - (STRICT ? 1 : 0)];
                    le &= __builtin_amdgcn_fcmpf(vm, fi[m], kUle);
                    if (!STRICT) lt |= __builtin_amdgcn_fcmpf(vm, fi[m], kOlt);
                }
                // a lone compare's mask takes the scalar path like the others:
                // a vector instruction may not read it straight from the compare
                if constexpr (STRICT && M == 2) asm("s_and_b64 %0, %0, exec" : "+s"(le) : : "scc");
                acc = shift_in(acc, STRICT ? le : le & lt);
            }
        }
        out[w] = acc;
    }
}

// Block (ic, jc): the points of chunk ic against the positions of chunk jc; one
// pair of chunks per block, since a block waits for the scalar loads of each
// batch of positions in turn, and few blocks of several chunks leave it at that:
// with four per block 2000 points of 8 objectives took 258 us in 16 blocks.  A
// generation of 1000 x 30 with 8 objectives, four / one: 390 / 182 us (counting
// over all pairs 324); 1000 x 100 with 3: 180 / 143; 16,384 x 100 with 3: 401 / 365;
// 16,384 x 100 with 8: 1488 / 1228.  The pointers are arguments of their own, marked unaliased, so that the
// positions' objectives (the same in every lane) come through scalar loads.
template <int M>
__global__ __launch_bounds__(kNsgaChunk) void k_nsga_bits(const float *__restrict__ fs,
                                                          const float *__restrict__ fr,
                                                          const float *__restrict__ range, int64_t n, int64_t chunks,
                                                          uint4 *__restrict__ W, uint32_t *__restrict__ ptr)
{
    const int64_t ic = blockIdx.x, jc = blockIdx.y, pos = ic * kNsgaChunk + threadIdx.x;
    constexpr int P = M <= 4 ? 4 : 8;
    if (!chunk_open(range, ic, jc)) return;
    float fi[M];
#pragma unroll
    for (int m = 0; m < M; ++m) fi[m] = fs[pos * P + m];
    uint32_t w[8];
    if (range[2 * jc + 1] < range[2 * ic])
        chunk_bits<M, true>(fr, jc, fi, w);
    else
        chunk_bits<M, false>(fs, jc, fi, w);
    if (pos >= n) return;
    W[w_index(chunks, ic, 2 * jc, threadIdx.x)] = make_uint4(w[0], w[1], w[2], w[3]);
    W[w_index(chunks, ic, 2 * jc + 1, threadIdx.x)] = make_uint4(w[4], w[5], w[6], w[7]);
    // the first group of four words with a dominator
    if (w[0] | w[1] | w[2] | w[3])
        atomicMin(ptr + pos, (uint32_t)(2 * jc));
    else if (w[4] | w[5] | w[6] | w[7])
        atomicMin(ptr + pos, (uint32_t)(2 * jc + 1));
}

// Fronts are found kNsgaPeelBatch at a time without a host round trip:
// lens[kb] counts front (k0 + kb) of the batch, the fronts before the batch
// hold `assigned0` points, and a front is only searched for while the points
// assigned before it are fewer than `need`.
__device__ __forceinline__ int64_t batch_base(const uint32_t *lens, int32_t kb, int64_t assigned0)
{
    int64_t base = assigned0;
    for (int32_t r = 0; r < kb; ++r) base += lens[r];
    return base;
}

constexpr int kFrontBlock = 512;

// Front k: the unassigned points with no unassigned dominator, appended to
// list.  A block has 64 positions; one thread each looks at the group its
// point waits on, then sixteen lanes each search the rows of the points that
// wait no more, 32 rows at a time (16 at a time: 14.3 us per front, 11.3 so).  The mask of unassigned points alternates between two buffers
// by the front's parity; a block writes the two words of its positions.
__global__ __launch_bounds__(kFrontBlock) void k_nsga_front(NsgaSortArgs a, int32_t k, int32_t kb, int64_t assigned0,
                                                    int64_t need)
{
    __shared__ __align__(16) uint32_t U[kNsgaMaxPoints / 32];
    __shared__ int32_t todo[64];
    __shared__ uint32_t ntodo, nmemb, at, memb[2];
    const int64_t base = batch_base(a.len, kb, assigned0);
    if (base >= need) return;  // the fronts needed are complete (uniform)
    const int tid = threadIdx.x, words = (int)(a.chunks * (kNsgaChunk / 32));
    const uint32_t *cur = a.mask + (k & 1) * words;
    for (int w = tid; w < words; w += kFrontBlock) U[w] = cur[w];
    if (tid == 0) ntodo = nmemb = 0;
    if (tid < 2) memb[tid] = 0;
    __syncthreads();
    const int64_t p0 = (int64_t)blockIdx.x * 64, ic = p0 / kNsgaChunk;
    const int pc = (int)(p0 % kNsgaChunk);
    auto blocked = [&](uint4 w, uint32_t g) {
        const uint4 u = *reinterpret_cast<const uint4 *>(U + 4 * g);
        return ((w.x & u.x) | (w.y & u.y) | (w.z & u.z) | (w.w & u.w)) != 0;
    };
    if (tid < 64 && p0 + tid < a.n && ((U[(p0 + tid) / 32] >> (31 - tid % 32)) & 1u)) {
        const uint32_t g = a.ptr[p0 + tid];
        if (g == kNsgaNoWord)
            atomicOr(&memb[tid / 32], 1u << (31 - tid % 32));
        else if (!blocked(a.W[w_index(a.chunks, ic, g, pc + tid)], g))
            todo[atomicAdd(&ntodo, 1u)] = tid;
    }
    __syncthreads();
    const int sub = tid / 16, l = tid % 16;
    const int groups = 2 * (int)a.chunks;
    for (uint32_t q = sub; q < ntodo; q += kFrontBlock / 16) {
        const int me = todo[q];
        uint32_t found = kNsgaNoWord;
        for (int g0 = (int)a.ptr[p0 + me] + 1; g0 < groups && found == kNsgaNoWord; g0 += 16) {
            const int g = g0 + l;
            const bool hit = g < groups && chunk_open(a.range, ic, g / 2) &&
                             blocked(a.W[w_index(a.chunks, ic, g, pc + me)], (uint32_t)g);
            const uint32_t b = (uint32_t)(__ballot(hit) >> (16 * (tid / 16 % 4))) & 0xffffu;
            if (b) found = (uint32_t)(g0 + __ffs((int)b) - 1);
        }
        if (l == 0) {
            a.ptr[p0 + me] = found;
            if (found == kNsgaNoWord) atomicOr(&memb[me / 32], 1u << (31 - me % 32));
        }
    }
    __syncthreads();
    if (tid == 0) {
        const uint32_t c = __popc(memb[0]) + __popc(memb[1]);
        at = c ? atomicAdd(a.len + kb, c) : 0u;
    }
    if (tid < 2) a.mask[((k & 1) ^ 1) * words + p0 / 32 + tid] = U[p0 / 32 + tid] & ~memb[tid];
    __syncthreads();
    if (tid < 64 && ((memb[tid / 32] >> (31 - tid % 32)) & 1u)) {
        // members before this one in the block
        const uint32_t before = (tid >= 32 ? __popc(memb[0]) : 0u) +
                                (tid % 32 ? __popc(memb[tid / 32] >> (32 - tid % 32)) : 0u);
        const int32_t i = a.ord[p0 + tid];
        a.front[i] = k;
        a.list[base + at + before] = i;
    }
}

// foff[k] = first list position of front k; foff[K] = total.
__global__ __launch_bounds__(256) void k_nsga_foff(const int32_t *list, int64_t total, const int32_t *front,
                                                   int32_t *foff)
{
    const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (q >= total) return;
    const int32_t k = front[list[q]];
    if (q == 0 || front[list[q - 1]] != k) foff[k] = (int32_t)q;
    if (q == total - 1) foff[k + 1] = (int32_t)total;
}

// Position of list entry q in each objective's order of (value, index)
// within its front: pos[m][q] += #{list entries r of the same front in this
// block's span : (F_r,m, r's point) < (F_q,m, q's point)}.  Fronts are
// contiguous in the list, so a block looks only at the part of its span
// inside its entries' fronts (and at the front numbers only when its entries
// lie in several); the work is the sum of the squared front sizes.  Bitwise
// comparisons, not short-circuit: no branch per entry.
template <int M>
__global__ __launch_bounds__(256) void k_nsga_order(NsgaSortArgs a, int64_t total)
{
    constexpr int P = M <= 4 ? 4 : 8;
    __shared__ __align__(16) float fj[kSpan * P];
    __shared__ int32_t ij[kSpan], kj[kSpan];
    const int64_t q0 = (int64_t)blockIdx.x * 256, r0 = (int64_t)blockIdx.y * kSpan;
    const int64_t qlast = q0 + 255 < total ? q0 + 255 : total - 1;
    const int32_t ka = a.front[a.list[q0]], kb = a.front[a.list[qlast]];
    const int64_t lo = a.foff[ka], hi = a.foff[kb + 1];
    const int64_t rb = r0 > lo ? r0 : lo, re = r0 + kSpan < hi ? r0 + kSpan : hi;
    if (rb >= re) return;
    const int nr = (int)(re - rb);
    for (int r = threadIdx.x; r < nr; r += 256) {
        const int32_t j = a.list[rb + r];
        ij[r] = j;
        kj[r] = a.front[j];
        load_pad<P>(fj + r * P, a.F, j, M);
    }
    __syncthreads();
    const int64_t q = q0 + threadIdx.x;
    if (q >= total) return;
    const int32_t i = a.list[q], k = a.front[i];
    float fi[M];
    int32_t c[M];
#pragma unroll
    for (int m = 0; m < M; ++m) {
        fi[m] = a.F[(int64_t)i * M + m];
        c[m] = 0;
    }
    auto count = [&](auto several) {
#pragma unroll 4
        for (int r = 0; r < nr; ++r) {
            const bool same = !several.value || kj[r] == k, below = ij[r] < i;
            float v[P];
#pragma unroll
            for (int h = 0; h < P / 4; ++h) {
                const float4 t = *reinterpret_cast<const float4 *>(fj + r * P + 4 * h);
                v[4 * h] = t.x, v[4 * h + 1] = t.y, v[4 * h + 2] = t.z, v[4 * h + 3] = t.w;
            }
#pragma unroll
            for (int m = 0; m < M; ++m) c[m] += (int32_t)(same & ((v[m] < fi[m]) | ((v[m] == fi[m]) & below)));
        }
    };
    if (ka == kb)
        count(std::false_type{});
    else
        count(std::true_type{});
#pragma unroll
    for (int m = 0; m < M; ++m)
        if (c[m]) atomicAdd(a.pos + m * a.cap + q, c[m]);
}

// sorted[m][foff[k] + pos[m][q]] = the point of list entry q.
__global__ __launch_bounds__(256) void k_nsga_scatter(NsgaSortArgs a, int64_t total)
{
    const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (q >= total) return;
    const int32_t i = a.list[q], b = a.foff[a.front[i]];
    for (int m = 0; m < a.M; ++m) a.sorted[m * a.cap + b + a.pos[m * a.cap + q]] = i;
}

// Crowding distance of list entry q: per objective in order, +inf at either
// end of the front's order, else + (next - previous) / (last - first) when
// the range is not zero (fp64).
__global__ __launch_bounds__(256) void k_nsga_crowd(NsgaSortArgs a, int64_t total)
{
    const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (q >= total) return;
    const int32_t i = a.list[q], k = a.front[i];
    const int32_t b = a.foff[k], e = a.foff[k + 1], size = e - b;
    double d = 0.0;
    for (int m = 0; m < a.M; ++m) {
        const int32_t p = a.pos[m * a.cap + q];
        const int32_t *srt = a.sorted + m * a.cap + b;
        if (p == 0 || p == size - 1) {
            d = INFINITY;
        } else {
            const double lo = (double)a.F[(int64_t)srt[0] * a.M + m];
            const double hi = (double)a.F[(int64_t)srt[size - 1] * a.M + m];
            if (hi > lo)
                d += ((double)a.F[(int64_t)srt[p + 1] * a.M + m] - (double)a.F[(int64_t)srt[p - 1] * a.M + m]) /
                     (hi - lo);
        }
    }
    a.crowd[i] = d;
    a.pos[q] = 0;  // the truncation counts its ranks here
}

// Rank of the last front's entry q (list positions [full, total)) in the
// order of (crowding descending, index): rank[q - full] += #{entries of this
// block's span ahead of it}.
__global__ __launch_bounds__(256) void k_nsga_trunc(const int32_t *list, int64_t full, int64_t total,
                                                    const double *crowd, int32_t *rank)
{
    __shared__ double cj[kSpan];
    __shared__ int32_t ij[kSpan];
    const int64_t size = total - full, r0 = (int64_t)blockIdx.y * kSpan;
    const int64_t nr = size - r0 < kSpan ? size - r0 : kSpan;
    for (int64_t r = threadIdx.x; r < nr; r += 256) {
        const int32_t j = list[full + r0 + r];
        ij[r] = j;
        cj[r] = crowd[j];
    }
    __syncthreads();
    const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (q >= size) return;
    const int32_t i = list[full + q];
    const double ci = crowd[i];
    int32_t c = 0;
    // bitwise, not short-circuit: no branch per entry, so the loop unrolls
#pragma unroll 8
    for (int64_t r = 0; r < nr; ++r) c += (int32_t)((cj[r] > ci) | ((cj[r] == ci) & (ij[r] < i)));
    if (c) atomicAdd(rank + q, c);
}

// keep[i] of every point: 1 for the survivors, the members of the fronts before
// the last and the last front's entries ranked below `need`.
__global__ __launch_bounds__(256) void k_nsga_keep(const int32_t *list, int64_t n, int64_t full, int64_t total,
                                                   int64_t need, const int32_t *rank, const int32_t *front,
                                                   int32_t *keep)
{
    const int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (q < total) keep[list[q]] = q < full || rank[q - full] < need ? 1 : 0;
    if (q < n && front[q] < 0) keep[q] = 0;  // in no front found
}

// Exclusive prefix sums of keep[0 .. n), by one block: rounds of four entries
// per thread, a wave scan each and the waves' sums through LDS.
__global__ __launch_bounds__(1024) void k_nsga_scan(const int32_t *keep, int64_t n, int32_t *pre)
{
    constexpr int R = kNsgaMaxPoints / 4096;
    __shared__ int32_t wsum[2][16];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int4 v[R];  // every round's entries (n is even: pairs are whole) in flight
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int64_t b = 4096 * r + 4 * threadIdx.x;
        v[r] = b + 3 < n ? *reinterpret_cast<const int4 *>(keep + b)
                         : b + 1 < n ? make_int4(keep[b], keep[b + 1], 0, 0) : make_int4(0, 0, 0, 0);
    }
    int32_t carry = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int64_t b = 4096 * r + 4 * threadIdx.x;
        if (4096 * (int64_t)r >= n) break;
        const int32_t s = v[r].x + v[r].y + v[r].z + v[r].w;
        int32_t inc = s;
        for (int d = 1; d < 64; d <<= 1) {
            const int32_t o = __shfl_up(inc, d, 64);
            if (lane >= d) inc += o;
        }
        if (lane == 63) wsum[r & 1][wave] = inc;  // alternating: no second barrier per round
        __syncthreads();
        int32_t run = carry + inc - s;
#pragma unroll
        for (int w = 0; w < 16; ++w) {
            const int32_t t = wsum[r & 1][w];
            run += w < wave ? t : 0;
            carry += t;
        }
        const int4 o = make_int4(run, run + v[r].x, run + v[r].x + v[r].y, run + v[r].x + v[r].y + v[r].z);
        if (b + 3 < n) {
            *reinterpret_cast<int4 *>(pre + b) = o;
        } else if (b + 1 < n) {
            pre[b] = o.x;
            pre[b + 1] = o.y;
        }
    }
}

// Survivor i of the merged population (parents 0..N-1, offspring N..2N-1)
// to row pre[i]: its row (float4 chunk c per thread), objectives, front and
// crowding distance.
__global__ __launch_bounds__(256) void k_nsga_compact(NsgaSelArgs a)
{
    const int64_t c4 = a.ldx / 4, q = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (q >= 2 * a.N * c4) return;
    const int64_t i = q / c4, c = q % c4;
    if (!a.keep[i]) return;
    const int64_t r = a.pre[i];
    const float *src = i < a.N ? a.X + i * a.ldx : a.Q + (i - a.N) * a.ldx;
    *reinterpret_cast<float4 *>(a.X2 + r * a.ldx + 4 * c) = *reinterpret_cast<const float4 *>(src + 4 * c);
    if (c == 0) {
        for (int m = 0; m < a.M; ++m) a.F[r * a.M + m] = a.FR[i * a.M + m];
        a.front[r] = a.frontR[i];
        a.crowd[r] = a.crowdR[i];
    }
}

__global__ __launch_bounds__(256) void k_fill_i32(int32_t *p, int64_t n, int32_t v)
{
    for (int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x; q < n; q += (int64_t)gridDim.x * 256) p[q] = v;
}

unsigned blocks(int64_t n, int64_t per) { return (unsigned)((n + per - 1) / per); }

#define EVOX_NSGA_M_SWITCH(M, CALL) \
    switch (M) {                   \
        case 2: CALL(2); break;    \
        case 3: CALL(3); break;    \
        case 4: CALL(4); break;    \
        case 5: CALL(5); break;    \
        case 6: CALL(6); break;    \
        case 7: CALL(7); break;    \
        case 8: CALL(8); break;    \
        default: return hipErrorInvalidValue; \
    }

}  // namespace

hipError_t launch_nsga_var(const NsgaVarArgs &a, hipStream_t s)
{
    const int64_t n = a.N / 2 * a.D;
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_nsga_var, dim3(blocks(n, 256)), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_nsga_dtlz1(const float *X, int64_t n, int64_t D, int64_t ldx, int32_t M, const float *Fold,
                             int64_t nold, float *F, uint32_t *hist, hipStream_t s)
{
    if (n == 0) return hipSuccess;
    const int64_t waves = n + (nold * M + 63) / 64;
    hipLaunchKernelGGL(k_nsga_dtlz1, dim3(blocks(waves, 4)), dim3(256), 0, s, X, n, D, ldx, M, Fold, nold, F, hist);
    return hipGetLastError();
}

hipError_t nsga_relate(const NsgaSortArgs &args, hipStream_t s)
{
    const int64_t n = args.n;
    if (n == 0) return hipSuccess;
    NsgaSortArgs a = args;
    a.chunks = (n + kNsgaChunk - 1) / kNsgaChunk;
    hipError_t e;
    hipLaunchKernelGGL(k_nsga_assign, dim3(blocks(n, 1024)), dim3(1024), 0, s, a.F, (int32_t)n, a.M, a.hist, a.ptr);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(k_nsga_place, dim3(blocks(n, 1024)), dim3(1024), 0, s, (int32_t)n, (const uint32_t *)a.hist,
                       (const uint32_t *)a.ptr, a.ord);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    const dim3 chunks((unsigned)a.chunks), grid((unsigned)a.chunks, (unsigned)a.chunks);
#define EVOX_RELATE(MM)                                                                                        \
    hipLaunchKernelGGL((k_nsga_gather<MM>), chunks, dim3(kNsgaChunk), 0, s, a);                                \
    hipLaunchKernelGGL((k_nsga_bits<MM>), grid, dim3(kNsgaChunk), 0, s, (const float *)a.Fs,         \
                       (const float *)a.Fr, (const float *)a.range, n, a.chunks, a.W, a.ptr)
    EVOX_NSGA_M_SWITCH(a.M, EVOX_RELATE)
#undef EVOX_RELATE
    return hipGetLastError();
}

hipError_t nsga_fronts(const NsgaSortArgs &args, int64_t need, NsgaSortResult *res, hipStream_t s)
{
    const int64_t n = args.n;
    *res = NsgaSortResult{0, 0, 0};
    if (n == 0) return hipSuccess;
    NsgaSortArgs a = args;
    a.chunks = (n + kNsgaChunk - 1) / kNsgaChunk;
    hipError_t e;
    int64_t assigned = 0, last = 0;
    int32_t k = 0;
    uint32_t lens[kNsgaPeelBatch];
    while (assigned < need) {
        if (k && (e = launch_zero_u32(a.len, kNsgaPeelBatch, s)) != hipSuccess) return e;  // the first: k_nsga_gather
        for (int32_t kb = 0; kb < kNsgaPeelBatch; ++kb) {
            hipLaunchKernelGGL(k_nsga_front, dim3((unsigned)a.chunks * (kNsgaChunk / 64)), dim3(kFrontBlock), 0, s, a, k + kb,
                               kb, assigned, need);
            if ((e = hipGetLastError()) != hipSuccess) return e;
        }
        if ((e = hipMemcpyAsync(lens, a.len, sizeof lens, hipMemcpyDeviceToHost, s)) != hipSuccess ||
            (e = hipStreamSynchronize(s)) != hipSuccess)
            return e;
        for (int32_t kb = 0; kb < kNsgaPeelBatch && assigned < need; ++kb) {
            if (lens[kb] == 0) return hipErrorUnknown;  // cannot happen: a finite set has a non-dominated point
            last = lens[kb];
            assigned += last;
            ++k;
        }
    }
    hipLaunchKernelGGL(k_nsga_foff, dim3(blocks(assigned, 256)), dim3(256), 0, s, (const int32_t *)a.list, assigned,
                       (const int32_t *)a.front, a.foff);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    const dim3 og(blocks(assigned, 256), blocks(assigned, kSpan));
#define EVOX_ORDER(MM) hipLaunchKernelGGL((k_nsga_order<MM>), og, dim3(256), 0, s, a, assigned)
    EVOX_NSGA_M_SWITCH(a.M, EVOX_ORDER)
#undef EVOX_ORDER
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(k_nsga_scatter, dim3(blocks(assigned, 256)), dim3(256), 0, s, a, assigned);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(k_nsga_crowd, dim3(blocks(assigned, 256)), dim3(256), 0, s, a, assigned);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    *res = NsgaSortResult{k, assigned, last};
    return hipSuccess;
}

hipError_t nsga_sort(const NsgaSortArgs &a, int64_t need, NsgaSortResult *res, hipStream_t s)
{
    hipError_t e = launch_zero_u32(a.hist, kNsgaSplit + 1, s);
    if (e != hipSuccess || (e = nsga_relate(a, s)) != hipSuccess) return e;
    return nsga_fronts(a, need, res, s);
}

hipError_t launch_nsga_select(const NsgaSelArgs &a, const NsgaSortResult &r, hipStream_t s)
{
    const int64_t full = r.assigned - r.last, need = a.N - full;
    hipError_t e;
    hipLaunchKernelGGL(k_nsga_trunc, dim3(blocks(r.last, 256), blocks(r.last, kSpan)), dim3(256), 0, s, a.list, full,
                       r.assigned, a.crowdR, a.rank);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(k_nsga_keep, dim3(blocks(2 * a.N, 256)), dim3(256), 0, s, a.list, 2 * a.N, full, r.assigned,
                       need, (const int32_t *)a.rank, a.frontR, a.keep);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(k_nsga_scan, dim3(1), dim3(1024), 0, s, (const int32_t *)a.keep, 2 * a.N, a.pre);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(k_nsga_compact, dim3(blocks(2 * a.N * (a.ldx / 4), 256)), dim3(256), 0, s, a);
    return hipGetLastError();
}

}  // namespace evox
