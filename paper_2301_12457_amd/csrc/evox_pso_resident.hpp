// A whole n-generation PSO call in one launch, the swarm resident on the chip.
//
// Between the evaluation of a generation and its move stands the global best.
// The grid-wide kernels (k_pso) cut the launch there and move the swarm through
// memory once per generation; for a swarm that fits in the registers and LDS
// of the 256 CUs (up to 10 million elements) both are avoidable.  Here a block
// keeps its rows -- x and pbest in registers, v in registers or LDS -- for the
// whole call, and the blocks agree on the global best once per generation
// through one 8-byte slot each:
//   - every block finds its best (pfit, row), stores that pbest row through to
//     memory if it changed, waits for the store, then stores its slot: the
//     value's 32 ordered bits, an 8-bit tag of the generation, 24 bits of index;
//   - every block reads all slots until each carries the tag (the slots are the
//     barrier: there is no counter to contend on), takes the minimum, and
//     fetches the winner's row if the winner changed.
// Slots and rows alternate between two buffers by the generation's parity: a
// block overwrites a buffer two generations later, after the exchange between
// in which every block has shown to be done with it.  All stores and loads that
// cross blocks are agent-scope atomics (written through, read past the caches),
// so no fence writes back an L2.  The number of exchanges is n_gens in every
// block, whatever the data.  The half of the move that does not need the global
// best runs between the store of the slot and the wait.
//
// The launch is cooperative: the grid fits the device.  That does not make the
// blocks start together -- a kernel of another stream or process may hold a CU
// for as long as it likes -- so a wait ends by the clock (PsoResArgs::wait) and
// the call is then given up and done by one block instead.  Nothing of the
// swarm is stored before the end of a call, so it only has to be decided once
// and for every block alike whether the call was completed, in ctl[0]:
//   - a block whose wait has run out turns kResRun into kResTry and, at the last
//     exchange, reads the slots again; if one is still missing, or at an earlier
//     exchange, it turns kResTry into kResAlone and leaves (else it goes on);
//   - a block that has passed the last exchange reads ctl[0]: kResRun and it
//     stores its rows (a block that tries later finds every slot); else it turns
//     kResTry into kResDone and stores, or finds kResAlone and leaves.
// One of the two changes of kResTry is made, and every block that finds the word
// changed follows it.  A block that read kResRun is never contradicted: kResAlone
// needs a slot of the last exchange missing after kResTry was set (the leaving
// block's own if it leaves earlier), and who sees all of them after that reads
// the word later still.  The usual call pays one
// read (a compare-and-swap by every block on one word cost 4 us a call).  After
// kResAlone every block leaves, those that start late as well, and the last one
// out (a count in ctl[1]) runs the whole call on the untouched swarm (pso_walk).
// The results are the same bits either way.
//
// One block (nblocks 1) needs none of this and is an ordinary launch.
//
// What bounds it: the exchange (two trips to memory, about 1.8 us with the
// arithmetic of small swarms), the vector ALU's issue rate for large ones
// (10,000 x 1000: 38 chunk waves per SIMD and generation) and for one block's (7
// waves on 4 SIMDs at 100 x 10).  A call of 25, 25, 20, 20 and 20 generations,
// against launches of k_pso or the one-block kernel it replaced: Sphere 100 x 10
// 61.2 -> 27.0 us, Rastrigin 1638 x 10 350 -> 69.5, Schwefel 1999 x 101 194 -> 73,
// Sphere 40,000 x 100 467 -> 190, Ackley 10,000 x 1000 860 -> 440.
#pragma once

#include "evox_kernels.hpp"

namespace evox {

constexpr uint64_t kResNoSlot = ~(uint64_t)0;  // tag 255, and generation 254's slots are not the first
// ctl[0] of a call; ctl[1] counts the blocks out, from -1 on (both words are
// all ones before a call, as its slots are)
constexpr uint32_t kResRun = 0xffffffffu, kResDone = 0, kResAlone = 1, kResTry = 2;

__device__ __forceinline__ uint32_t tag_of(uint64_t slot) { return ((uint32_t)slot >> 24) & 0xffu; }

// Keeps a value that does not change between generations from being carried
// through the generation loop in every form the compiler can derive from it.
// Scalar where the group is at least a wave.
template <int G>
__device__ __forceinline__ uint32_t opaque(uint32_t v)
{
    if constexpr (G >= 64) {
        v = (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
        asm volatile("" : "+s"(v));
    } else {
        asm volatile("" : "+v"(v));
    }
    return v;
}

// The kernel argument at the given offset, as a value of its own to the compiler.
template <typename V>
__device__ __forceinline__ V kernel_argument(uint32_t offset)
{
    typedef const __attribute__((address_space(4))) uint32_t *Words;
    uint64_t at = (uint64_t)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(at));
    Words src = (Words)(at + offset);
    uint32_t w[sizeof(V) / 4];
#pragma unroll
    for (uint32_t q = 0; q < sizeof(V) / 4; ++q) w[q] = src[q];
    V v;
    __builtin_memcpy(&v, w, sizeof v);
    return v;
}

// A whole n_gens-generation call by one block, the swarm in memory: per
// generation one walk over the rows to evaluate (the fitness bits of
// row_fitness) and one to move them.  nbr, red: LDS as row_fitness takes it;
// sk, sc: blockDim / 64 entries; sel: one; gb: 8 G floats.  The chunks of the move are not
// unrolled: both at once cost the resident kernel that this is a part of 60
// spilled registers in its ten-row shape.
template <int FN, int G>
__device__ __forceinline__ void pso_walk(const PsoArgs &a, int64_t n_gens, float *gbest_out, DevBest *best, float *nbr, float *red,
                         uint64_t *sk, uint32_t *sc, int64_t *sel, float *gb)
{
    constexpr int MAXIT = 2;
    const int tid = (int)opaque<1>(threadIdx.x), nt = blockDim.x, g = tid % G, slot = tid / G, gpb = nt / G;
    const uint32_t C4 = (uint32_t)((a.D + 3) >> 2);
    const uint32_t CW = (uint32_t)(a.ldx / 4 < G * MAXIT ? a.ldx / 4 : G * MAXIT);
    const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int64_t k = 0; k < n_gens; ++k) {
        uint64_t key = kNoKey;
        uint32_t nimp = 0;
        for (int64_t rb = 0; rb < a.N; rb += gpb) {  // uniform trip count: row_fitness has barriers
            const int64_t row = rb + slot;
            const bool active = row < a.N;
            const float pold = active ? a.pf[row] : 0.0f;
            float4 xr[MAXIT];
#pragma unroll
            for (int it = 0; it < MAXIT; ++it) {
                const uint32_t c = g + G * it;
                xr[it] = active && c < C4 ? *reinterpret_cast<const float4 *>(a.x + row * a.ldx + 4 * c) : zero;
            }
            const float f = row_fitness<FN, G, MAXIT>(xr, g, a.D, nbr, red);
            if (active) {
                const bool imp = f < pold;
                if (imp) {
#pragma unroll
                    for (int it = 0; it < MAXIT; ++it) {
                        const uint32_t c = g + G * it;
                        if (c < CW) *reinterpret_cast<float4 *>(a.p + row * a.ldx + 4 * c) = xr[it];
                    }
                }
                if (g == 0) {
                    if (imp) a.pf[row] = f;
                    if (a.fit) a.fit[row] = f;
                    const uint64_t kr = sel_key(imp ? f : pold, row);
                    key = kr < key ? kr : key;
                    nimp += imp ? 1u : 0u;
                }
            }
        }
        block_min_key(key, nimp, sk, sc);
        if (tid == 0) {
            best->f = key_value(key);
            best->i = *sel = key_index(key);
            best->improved += nimp;
        }
        __syncthreads();
        for (int64_t j = tid; j < a.ldx; j += nt) {
            const float t = a.p[*sel * a.ldx + j];
            gbest_out[j] = t;
            if (j < 4 * G * MAXIT) gb[j] = t;
        }
        __syncthreads();
        for (int64_t rb = 0; rb < a.N; rb += gpb) {
            const int64_t row = rb + slot;
#pragma unroll 1
            for (int it = 0; it < MAXIT; ++it) {
                const uint32_t c = g + G * it;
                const int64_t off = row * a.ldx + 4 * c;
                float4 xn = zero, vn = zero;
                if (row < a.N && c < C4) {
                    const float4 xv = *reinterpret_cast<const float4 *>(a.x + off);
                    const float4 pull =
                        pso_pull4(a, (uint32_t)row, c, a.t + (uint32_t)k, xv, *reinterpret_cast<const float4 *>(a.v + off),
                                  *reinterpret_cast<const float4 *>(a.p + off));
                    pso_push4<true, true>(a, c, pso_draw4(a, (uint32_t)row, c, a.t + (uint32_t)k), xv, pull,
                                          *reinterpret_cast<const float4 *>(gb + 4 * c), xn, vn);
                }
                if (row < a.N && c < CW) {
                    *reinterpret_cast<float4 *>(a.x + off) = xn;
                    *reinterpret_cast<float4 *>(a.v + off) = vn;
                }
            }
        }
        __syncthreads();  // the next generation evaluates every moved row
    }
}

// R rows per lane group of G lanes, two chunks per lane; VL of the R velocity
// rows in LDS, the rest in registers; at most T threads per block (T exactly
// when VL > 0).  MANY: more than one block (in one kernel with the other the
// scalar registers of either spill into the generation loop of both).
template <int FN, int G, int R, int VL, int T, bool MANY>
__global__ __launch_bounds__(T) void k_pso_res(PsoArgs a, PsoResArgs e)
{
    using F = Fn<FN>;
    constexpr int MAXIT = 2, NW = T / 64, VR = R - VL;
    constexpr bool SPAN = G > 64;  // a row spans several waves
    __shared__ float4 vls[VL > 0 ? VL * MAXIT * T : 1];
    // one block: each unit's (wave's, or spanning row's) best row by parity;
    // else the global best row
    constexpr bool ONE = R == 1;
    static_assert(MANY || R <= 3, "one block: up to three rows per group");
    constexpr int UNIT = G > 64 ? G : 64, NU = MANY ? 1 : 2 * (T / UNIT);
    __shared__ __align__(16) float gb[NU][G * MAXIT * 4];
    __shared__ uint64_t sk[2][NW], sm[NW];
    __shared__ Acc red[SPAN ? R : 1][NW];
    __shared__ float first[SPAN && F::kNeighbour ? R : 1][MAXIT][NW];
    __shared__ int32_t bad, lost, last;  // a wait ran out; the call is given up; the last block out
    __shared__ int64_t pick;

    const int tid = threadIdx.x, nt = blockDim.x, nw = nt / 64, lane = tid & 63, wave = tid >> 6;
    const int g = tid % G, slot = tid / G, gpb = nt / G;  // groups per block
    const int nb = MANY ? e.nblocks : 1, b = MANY ? blockIdx.x : 0;
    const uint32_t C4 = (uint32_t)((a.D + 3) >> 2);
    const uint32_t CW = (uint32_t)(a.ldx / 4 < G * MAXIT ? a.ldx / 4 : G * MAXIT);
    const uint32_t N = (uint32_t)a.N;
    const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
    // row r of the group: row0 + r step; the block has such rows at all when
    // live(r) (uniform).  Groups past the last row and lanes past a row's end
    // compute on zeros; nothing of theirs is selected or stored
    const uint32_t row0 = (uint32_t)(b * gpb + slot), step = (uint32_t)(nb * gpb);
    const bool clamp = a.vclamp || a.xclamp;  // uniform
    auto live = [&](int r) { return opaque<64>((uint32_t)(b * gpb)) + r * step < N; };  // compared anew: no masks kept

    float4 x[R][MAXIT], p[R][MAXIT], vr[VR > 0 ? VR : 1][MAXIT];
    float pf[R];
    auto getv = [&](int r, int it) { return r < VL ? vls[(r * MAXIT + it) * T + tid] : vr[r < VL ? 0 : r - VL][it]; };
    auto setv = [&](int r, int it, float4 v) {
        if (r < VL)
            vls[(r * MAXIT + it) * T + tid] = v;
        else
            vr[r < VL ? 0 : r - VL][it] = v;
    };
    // elements past D are zero from here on, whatever the padding holds
    auto keep = [&](float4 t, bool ld, uint32_t c) {
        const int left = ld ? (int)a.D - (int)(4 * c) : 0;
        return make_float4(left > 0 ? t.x : 0.0f, left > 1 ? t.y : 0.0f, left > 2 ? t.z : 0.0f, left > 3 ? t.w : 0.0f);
    };
    if constexpr (R <= 3) {
        // few rows: all their loads in flight together, unconditional (the last
        // row and chunk past the end)
        float4 vt[R][MAXIT];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const uint32_t row = row0 + r * step < N ? row0 + r * step : N - 1;
            pf[r] = a.pf[row];
#pragma unroll
            for (int it = 0; it < MAXIT; ++it) {
                const uint32_t c = g + G * it;
                const int64_t off = (int64_t)row * a.ldx + 4 * (c < C4 ? c : C4 - 1);
                x[r][it] = *reinterpret_cast<const float4 *>(a.x + off);
                p[r][it] = *reinterpret_cast<const float4 *>(a.p + off);
                vt[r][it] = *reinterpret_cast<const float4 *>(a.v + off);
            }
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const bool in = row0 + r * step < N;
            pf[r] = in ? pf[r] : 0.0f;
#pragma unroll
            for (int it = 0; it < MAXIT; ++it) {
                x[r][it] = keep(x[r][it], in, g + G * it);
                p[r][it] = keep(p[r][it], in, g + G * it);
                setv(r, it, keep(vt[r][it], in, g + G * it));
            }
        }
    } else {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const uint32_t row = row0 + r * step;
            const bool in = row < N;
            __builtin_amdgcn_sched_barrier(0);
            pf[r] = in ? a.pf[row] : 0.0f;
#pragma unroll
            for (int it = 0; it < MAXIT; ++it) {
                const uint32_t c = g + G * it;
                const int64_t off = (int64_t)row * a.ldx + 4 * c;
                const bool ld = in && c < C4;
                auto row4 = [&](const float *src) {
                    return keep(ld ? *reinterpret_cast<const float4 *>(src + off) : zero, true, c);
                };
                x[r][it] = row4(a.x);
                p[r][it] = row4(a.p);
                setv(r, it, row4(a.v));
            }
        }
    }
    const int looks = (int)opaque<64>((uint32_t)e.polls);  // in a register: not loaded at every poll
    const int64_t n_gens = MANY && e.wait == 0 ? 0 : e.n_gens;  // 0: given up at once
    if (tid == 0) {
        bad = MANY && e.wait == 0;
        lost = 0;
        if (MANY && e.wait == 0) store_through(e.ctl, kResAlone);
    }
    uint64_t win = kNoKey, sent[2] = {kNoKey, kNoKey};  // last winner; block bests whose rows the buffers hold
    uint32_t nimp = 0;
    const float4 *gsrc = reinterpret_cast<const float4 *>(gb[0]);
    __syncthreads();

    for (int64_t k = 0; k < n_gens; ++k) {
        const uint32_t t = a.t + (uint32_t)k;
        const int q = (int)(k & 1);
        // fitness of every row in the order of row_fitness, personal bests,
        // and the block's best (value, row)
        uint64_t key = kNoKey;
        const uint32_t rowe = opaque<G>(row0);
        auto decide = [&](int r, Acc s) {
            const uint32_t row = rowe + r * step;
            const float f = F::finish(s, a.D);
            const bool in = row < N, imp = in && f < pf[r];
            pf[r] = imp ? f : pf[r];
            nimp += imp && g == 0 ? 1u : 0u;
#pragma unroll
            for (int it = 0; it < MAXIT; ++it)
                if (imp) p[r][it] = x[r][it];
            if (k == n_gens - 1 && in && g == 0 && a.fit) a.fit[opaque<1>(row)] = f;
            const uint64_t kr = in ? sel_key(pf[r], row) : kNoKey;
            key = kr < key ? kr : key;
        };
        if constexpr (SPAN && F::kNeighbour) {
            if (lane == 0) {
#pragma unroll
                for (int r = 0; r < R; ++r)
#pragma unroll
                    for (int it = 0; it < MAXIT; ++it) first[r][it][wave] = x[r][it].x;
            }
            __syncthreads();
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (!live(r)) continue;
            float nbv[MAXIT] = {0.0f, 0.0f};
            if constexpr (F::kNeighbour) {
#pragma unroll
                for (int it = 0; it < MAXIT; ++it) {
                    if constexpr (!SPAN) {
                        const float same = __shfl(x[r][it].x, (g + 1) & (G - 1), G);
                        const float next = it + 1 < MAXIT ? __shfl(x[r][it + 1 < MAXIT ? it + 1 : it].x, 0, G) : 0.0f;
                        nbv[it] = g == G - 1 ? next : same;
                    } else {
                        // lane 63: the next wave's first element, or in the
                        // row's last wave the next chunk of its first
                        const float same = __shfl(x[r][it].x, (lane + 1) & 63, 64);
                        float edge = 0.0f;
                        if (lane == 63 && g != G - 1)
                            edge = first[r][it][wave + 1];
                        else if (lane == 63 && it + 1 < MAXIT)
                            edge = first[r][it + 1 < MAXIT ? it + 1 : it][wave - (G / 64 - 1)];
                        nbv[it] = lane == 63 ? edge : same;
                    }
                }
            }
            Acc s = row_partial<FN, G, MAXIT, true>(x[r], nbv, g, a.D);
            s = lanes_combine<FN, (SPAN ? 64 : G) / 2>(s);
            if constexpr (SPAN) {
                if (lane == 0) red[r][wave] = s;
            } else {
                decide(r, s);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (SPAN) {
            __syncthreads();
            constexpr int W = G / 64;
            const int w0 = wave / W * W;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if (!live(r)) continue;
                Acc s = red[r][w0];
#pragma unroll
                for (int u = 1; u < W; ++u) s = F::combine(s, red[r][w0 + u]);
                decide(r, s);
            }
        }
        const uint64_t own = key;
        if constexpr (G < 64) key = lanes_min<32, G>(key);
        if (lane == 0) sk[q][wave] = key;
        if constexpr (!MANY)
            if (own == key && key != kNoKey) {
                float4 *dst = reinterpret_cast<float4 *>(gb[q * (T / UNIT) + tid / UNIT]);
#pragma unroll
                for (int r = 0; r < R; ++r)
                    if (row0 + r * step == (uint32_t)key) {
#pragma unroll
                        for (int it = 0; it < MAXIT; ++it) dst[g + G * it] = p[r][it];
                    }
            }
        // the half of the move that needs no global best, before the wait for
        // the other waves (one row per group: both halves' random numbers) or
        // blocks: v <- fma(c1 r1, p - x, w v)
        float4 draw[ONE ? MAXIT : 1];
        auto pull = [&]() {
            const uint32_t ro = opaque<G>(row0), co = opaque<1>((uint32_t)g);
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if (!live(r)) continue;
#pragma unroll
                for (int it = 0; it < MAXIT; ++it)
                    if ((uint32_t)(G * it) < C4) {
                        setv(r, it, pso_pull4(a, ro + r * step, co + G * it, t, x[r][it], getv(r, it), p[r][it]));
                        if constexpr (ONE) draw[it] = pso_draw4(a, ro, co + G * it, t);
                    }
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        if constexpr (!MANY) pull();
        __syncthreads();
        key = lanes_min<8>(sk[q][(lane & 15) < nw ? lane & 15 : 0]);
        if constexpr (MANY) {
            const bool fresh = key != sent[q];  // uniform over the block
            sent[q] = key;
            if (fresh) {
                const uint32_t best = (uint32_t)key;
                uint64_t *dst = e.cand + ((int64_t)q * nb + b) * (G * MAXIT * 2);
#pragma unroll
                for (int r = 0; r < R; ++r)
                    if (row0 + r * step == best && key != kNoKey) {
#pragma unroll
                        for (int it = 0; it < MAXIT; ++it) {
                            const uint64_t *src = reinterpret_cast<const uint64_t *>(&p[r][it]);
                            store_through(dst + 2 * (g + G * it), src[0]);
                            store_through(dst + 2 * (g + G * it) + 1, src[1]);
                        }
                    }
                wait_stores();
                __syncthreads();
            }
            // value | tag | index; a block without rows sends the largest value
            const uint64_t tag = (uint64_t)((uint32_t)(k + 1) & 0xffu) << 24;
            if (tid == 0)
                store_through(e.slots + q * nb + b, (key & ~(uint64_t)0xffffffffu) | tag | (key & 0xffffffu));
        }
        if constexpr (MANY) {
            pull();
            const uint32_t want = (uint32_t)(k + 1) & 0xffu;
            uint64_t m = kNoKey;
            if (__builtin_amdgcn_readfirstlane(wave) * 64 < nb) {
                // slots tid, tid + nt, ... (the last one again past the end): all
                // loads of a poll in flight, the wave's loop on scalar branches
                constexpr int P = kResBlocks / 64;
                uint64_t w[P];
                const uint64_t *base = e.slots + q * nb;
                const bool one = nt >= nb;
                auto poll = [&] {
                    if (!one) {
#pragma unroll
                        for (int u = 1; u < P; ++u) w[u] = load_past(base + (tid + u * nt < nb ? tid + u * nt : nb - 1));
                    }
                    w[0] = load_past(base + (tid < nb ? tid : nb - 1));
                    bool all = tag_of(w[0]) == want;
                    if (!one) {
#pragma unroll
                        for (int u = 1; u < P; ++u) all &= tag_of(w[u]) == want;
                    }
                    return __ballot(!all) == 0;
                };
                uint64_t since = 0;
                for (;;) {
                    bool all;
                    int polls = 0;
                    do all = poll();
                    while (!all && ++polls < looks);
                    if (__builtin_expect(all, 1)) break;
                    const uint64_t now = wall_clock64();
                    if (since == 0) since = now;
                    uint32_t st = __builtin_amdgcn_readfirstlane(load_past(e.ctl));
                    if ((st == kResRun || st == kResTry) && now - since >= e.wait) {
                        if (lane == 0) atomicCAS(e.ctl, kResRun, kResTry);
                        wait_stores();  // the word is set before the slots are read again
                        if (k == n_gens - 1 && poll()) break;
                        if (lane == 0) st = atomicCAS(e.ctl, kResTry, kResAlone) == kResDone ? kResDone : kResAlone;
                        st = __builtin_amdgcn_readfirstlane(st);
                    }
                    if (st == kResAlone) {
                        bad = 1;
                        break;
                    }
                }
                m = w[0];
                if (!one) {
#pragma unroll
                    for (int u = 1; u < P; ++u) m = w[u] < m ? w[u] : m;
                }
            }
            m = lanes_min<32>(m);
            if (lane == 0) sm[wave] = m;
            __syncthreads();
            key = lanes_min<8>(sm[(lane & 15) < nw ? lane & 15 : 0]);
            if (bad) break;  // uniform: written before the barrier
            key &= ~(uint64_t)0xff000000u;  // the tag out, the index back
        }
        if constexpr (!MANY) {
            uint32_t group = (uint32_t)key;
#pragma unroll
            for (int r = 1; r < R; ++r) group -= group >= step ? step : 0;
            gsrc = reinterpret_cast<const float4 *>(gb[q * (T / UNIT) + group * G / UNIT]);
        } else if (key != win) {
            const uint64_t *src =
                e.cand + ((int64_t)q * nb + (uint32_t)key / (uint32_t)gpb % (uint32_t)nb) * (G * MAXIT * 2);
            for (int j = tid; j < G * MAXIT * 2; j += nt) reinterpret_cast<uint64_t *>(gb[0])[j] = load_past(src + j);
            __syncthreads();
        }
        win = key;
        // the other half: vn = fma(c2 r2, g - x, v), the clamps, x + vn
        {
            const uint32_t ro = opaque<G>(row0), co = opaque<1>((uint32_t)g);
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if (!live(r)) continue;
#pragma unroll
                for (int it = 0; it < MAXIT; ++it)
                    if ((uint32_t)(G * it) < C4) {
                        float4 d, xn, vn;
                        if constexpr (ONE)
                            d = draw[it];
                        else
                            d = pso_draw4(a, ro + r * step, co + G * it, t);
                        if (clamp)
                            pso_push4<true, true>(a, co + G * it, d, x[r][it], getv(r, it), gsrc[g + G * it], xn, vn);
                        else
                            pso_push4<false, false>(a, co + G * it, d, x[r][it], getv(r, it), gsrc[g + G * it], xn, vn);
                        x[r][it] = xn;
                        setv(r, it, vn);
                    }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        // LDS is reused across generations without a barrier of its own: sk
        // (and one block's gb) alternate by parity, and first, red, sm and
        // gb are next written behind a barrier that every wave reaches after
        // its last read here
    }
    if constexpr (MANY) {
        // the other launch parity's words, idle now, are cleared for the next call
        if (tid < 2) {
            store_through(e.slots_next + tid * nb + b, kResNoSlot);
            if (b == 0) store_through(e.ctl_next + tid, kResRun);
        }
        // past the last exchange
        if (tid == 0 && !bad && load_past(e.ctl) != kResRun)
            lost = atomicCAS(e.ctl, kResTry, kResDone) == kResAlone;
        __syncthreads();
        // the same in every block; scalar branches, so that the rows are dead in it
        if (__builtin_amdgcn_readfirstlane(bad | lost)) {
            if (tid == 0) last = atomicAdd(e.ctl + 1, 1u) + 1u == (uint32_t)(nb - 1);
            __syncthreads();
            if (__builtin_amdgcn_readfirstlane(last)) {
                // fit may hold values of this call's last generation: those that
                // the walk stores again
                if (tid == 0) ++e.best->alone;
                float *nbr = nullptr;
                if constexpr (SPAN && F::kNeighbour) {
                    __shared__ float own[VL > 0 ? 1 : T * MAXIT];
                    nbr = VL > 0 ? reinterpret_cast<float *>(vls) : own;
                }
                // the arguments read again: none is carried here through the loop
                const PsoArgs wa = kernel_argument<PsoArgs>(0);
                const PsoResArgs we = kernel_argument<PsoResArgs>(sizeof(PsoArgs));
                pso_walk<FN, G>(wa, we.n_gens, we.gbest_out, we.best, nbr, reinterpret_cast<float *>(red), sk[0],
                                reinterpret_cast<uint32_t *>(sm), &pick, gb[0]);
            }
            return;
        }
    }

    {
        // opaque: the addresses are not carried through the loop from the loads
        const uint32_t ro = opaque<G>(row0), co = opaque<1>((uint32_t)g);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const uint32_t row = ro + r * step;
            if (row0 + r * step < N) {
#pragma unroll
                for (int it = 0; it < MAXIT; ++it) {
                    const uint32_t c = co + G * it;
                    const int64_t off = (int64_t)row * a.ldx + 4 * c;
                    if (c < CW) {
                        *reinterpret_cast<float4 *>(a.x + off) = x[r][it];
                        *reinterpret_cast<float4 *>(a.v + off) = getv(r, it);
                        *reinterpret_cast<float4 *>(a.p + off) = p[r][it];
                    }
                }
                if (g == 0) a.pf[row] = pf[r];
            }
        }
    }
    nimp = lanes_sum<32>(nimp);
    if (lane == 0 && nimp) atomicAdd((unsigned long long *)&e.best->improved, (unsigned long long)nimp);
    if (b == 0) {
        for (int j = tid; j < a.ldx; j += nt) e.gbest_out[j] = j < G * MAXIT * 4 ? reinterpret_cast<const float *>(gsrc)[j] : 0.0f;
        if (tid == 0) {
            e.best->f = key_value(win);
            e.best->i = key_index(win);
        }
    }
}

// The shapes (PsoResPlan::shape): one row per group with up to 1024 threads; 4
// rows with 512; three rows with up to 1024 in one block; 10 rows with 512 threads, x and pbest in 160 of
// the 256 registers that leaves a lane and v in LDS but for what the row of gb
// takes.
template <int FN, int G>
hipError_t launch_pso_res_g(const PsoResPlan &pl, PsoArgs &a, PsoResArgs &e, hipStream_t s)
{
    constexpr int VL = G == 512 ? 8 : 9;
    void *args[] = {&a, &e};
    if (pl.shape == 4) {
        if constexpr (G <= 64)
            return hipLaunchKernel(reinterpret_cast<const void *>(&k_pso_res<FN, G, 3, 0, 1024, false>), dim3(1),
                                   dim3((unsigned)pl.threads), args, 0, s);
        return hipErrorInvalidValue;
    }
    if (e.nblocks == 1)
        return hipLaunchKernel(reinterpret_cast<const void *>(&k_pso_res<FN, G, 1, 0, 1024, false>), dim3(1),
                               dim3((unsigned)pl.threads), args, 0, s);
    const void *f = pl.shape == 1   ? reinterpret_cast<const void *>(&k_pso_res<FN, G, 1, 0, 1024, true>)
                    : pl.shape == 2 ? reinterpret_cast<const void *>(&k_pso_res<FN, G, 4, 0, 512, true>)
                                    : reinterpret_cast<const void *>(&k_pso_res<FN, G, 10, VL, 512, true>);
    return hipLaunchCooperativeKernel(f, dim3((unsigned)e.nblocks), dim3((unsigned)pl.threads), args, 0, s);
}

template <int FN>
hipError_t launch_pso_res_t(int G, const PsoResPlan &pl, const PsoArgs &args, const PsoResArgs &eargs, hipStream_t s)
{
    PsoArgs a = args;
    PsoResArgs e = eargs;
    switch (G) {
        case 4: return launch_pso_res_g<FN, 4>(pl, a, e, s);
        case 8: return launch_pso_res_g<FN, 8>(pl, a, e, s);
        case 16: return launch_pso_res_g<FN, 16>(pl, a, e, s);
        case 32: return launch_pso_res_g<FN, 32>(pl, a, e, s);
        case 64: return launch_pso_res_g<FN, 64>(pl, a, e, s);
        case 128: return launch_pso_res_g<FN, 128>(pl, a, e, s);
        case 256: return launch_pso_res_g<FN, 256>(pl, a, e, s);
        case 512: return launch_pso_res_g<FN, 512>(pl, a, e, s);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace evox
