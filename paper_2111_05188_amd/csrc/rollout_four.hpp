// Rollout kernel for actors outside the role-split kernel's shapes: fp32 ones
// with hidden widths to 1,024, bf16 ones as rollout_four_shape says.  One launch
// runs all L lockstep steps of 4, 8 or (bf16) 16 envs per workgroup.
//
// What bounds such a rollout is the chain of one step: a small market and a
// small actor leave little work, and every step is layer 1 -> 2 -> 3 -> env
// step.  Three things shorten it:
//
//  - MFMAs without padding of 4 envs.  fp32: v_mfma_f32_4x4x1_16b_f32
//    multiplies sixteen 4 x 4 blocks.  Four blocks take the 16 outputs of a
//    tile, and four such sets a quarter of the inputs each, with fragments in
//    the layout of the 16 x 16 MFMAs; the quarters meet by lane swaps that leave
//    one (output, env) a lane for the bias and the tanh.  bf16: the 16 columns
//    of v_mfma_f32_16x16x32_bf16 repeat the envs, and each lane finishes its
//    share of its four outputs.
//  - Weights that stay.  The LDS that rows and activations leave free is
//    filled with weights once per launch (the action layer first, then the
//    state columns of layer 1, layer 2, the market columns), and the matrix
//    waves keep some of layer 2 in registers; only the rest
//    streams from L2, a few k-blocks ahead.
//  - Roles.  Four matrix waves compute the layers.  A trade wave per four
//    envs (16 lanes an env, env_row.hpp) runs the env step and an aux wave
//    everything beside the chain: market rows, normals, observation rows.
//    The market columns of layer 1 are multiplied while the trade runs.
//
// An output's sum takes its k-blocks in the same order for 4, 8 and 16 envs a
// workgroup, whichever of them are resident, so the split does not show in the
// results.
//
// Per step j, separated by workgroup barriers:
//
//   slot  matrix waves                    trade wave          aux wave
//   A     z = W1[:, market] x_j           env step j-1 (the   normals of step j, market
//                                         state columns of    columns of x_{j+1} into
//                                         x_j)                x_{j-1}'s place
//   B     h1 = tanh(z + W1[:, state] x_j + b1)
//   L2    h2 = tanh(W2 h1 + b2)                               trajectory row j-1
//   L3    mu = W3 h2 + b3                                     x_j to HBM, loads of row j+2
//
// Measured (us per lockstep step, generic kernel -> this one; whole CUs
// streaming): 64 envs of 31-64-64-5 fp32 9.2 -> 2.5; 1,024 envs of
// 301-256-256-30 fp32 17.5 -> 7.7; 1,332 of it in bf16 13.0 -> 4.9; 16,384 envs
// of 31-64-64-5 78 -> 23.  At 31-64-64-5 the trade bounds slot A (2,100 of
// 5,700 cycles), latencies the others.  At 301-256-256-30 fp32 loads do: 390 KB a
// step at the CU's 64 bytes a cycle are 6,000 of 17,500 cycles, and a wave
// that issues them waits for the ones before.  What helped there: no global
// access in the trade (a store queues behind the weights), registers beside the
// LDS, N = 4 MFMAs, finishing tiles without conditions (their chains then
// interleave).  Spreading a layer's first loads over the layer before: nothing.
//
// Rows in LDS are observation rows.  A k-block is 64 bytes of inputs: 16 fp32
// or 32 bf16.  Layer 1's state blocks hold the balance or a holding, the
// others (market blocks) only prices and indicators.
#pragma once

#include <type_traits>

#include "device.hpp"
#include "env_row.hpp"
#include "internal.hpp"

namespace tpk {
namespace four {

constexpr int MW = 4;       // matrix waves

typedef uint32_t u4v __attribute__((ext_vector_type(4)));

template <int I>
using ic = std::integral_constant<int, I>;

// One layer (or part of one): nt tiles of 16 outputs, kb of the layer's KB
// k-blocks of 64 bytes of inputs: its block k is the layer's block first + k,
// from `cut` on first + skip + k.  Weights as fragments [nt][KB][64 lanes][16
// bytes] at `off` of the agent's packed buffer; the first `res` blocks of
// every tile also in LDS, [nt][res][1 KiB] at `lds`.
struct Part {
    int out, nt, kb, KB, first, cut, skip, res, lds, off;
};

struct Plan {
    Part part[4];           // layer 1 market, layer 1 state, layer 2, layer 3
    int ldx, ldh1, ldh2;    // byte pitches
    int ldm;                // stock slots per env (16 N)
    int X, H1, H2, MU, SZ, PN, LP, RW, BIAS, bytes;
};

// k-blocks of layer 2 a matrix wave keeps in registers for its first GT
// tiles (4 GT registers each), and k-blocks in flight for G tiles
constexpr int keep_blocks(int GT, int NG, int TW)
{
    const int r = (TW == 4 || NG == 4 ? 4 : NG == 1 ? 24 : 16) / GT;
    return r > 8 ? 8 : r;
}
constexpr int flight(int G) { return G <= 2 ? 8 : 4; }   // even: inputs take turns

template <bool BF>
struct Elem {
    typedef float T;
};
template <>
struct Elem<true> {
    typedef __bf16 T;
};

template <bool BF>
__device__ __forceinline__ typename Elem<BF>::T cvt(float x)
{
    return (typename Elem<BF>::T)x;
}

// Input fragments and accumulators per tile: fp32 one for every four envs, bf16
// one for all.
template <bool BF, int NG>
constexpr int XS = BF ? 1 : NG;

// Accumulators of G tiles.  fp32: two each for one tile at a time (narrow
// networks and the action layer), the even and the odd elements of every
// lane's 16 bytes, so eight partial sums an output: the sums of short layers
// are then no further from 64 bits than those of the VALU layers of fp32
// actors over 1,024 wide, which are split over as many lanes.
template <bool BF, int G>
constexpr int ACCS = !BF && G == 1 ? 2 : G;

// acc += one k-block of G tiles (w) against the envs' inputs (x).  Lane l
// holds 16 bytes of inputs kq = l / 16 of the block: in w those of output
// l % 16, in x those of env l % 4 (bf16: of env l % MB).
// fp32: block b = l / 4 of the MFMA multiplies four outputs by four envs, so
// lane l sums output l % 16 over its kq, for the four envs in its four
// registers.  bf16: one 16 x 16 x 32 MFMA, its 16 columns the MB envs over and
// over, so lane l has outputs 4 (l / 16) .. + 3 of env l % MB.  (It does the
// work of four 4 x 4 x 4 ones in half their cycles where MB = 8, and leaves
// nothing to sum over lanes: 1,332 envs of 301-256-256-30 1,442 -> 1,268 us.)
template <bool BF, int NX, int G>
__device__ __forceinline__ void block(const u4v *w, const u4v *x, floatx4 (&acc)[ACCS<BF, G>][NX])
{
    if constexpr (BF) {
#pragma unroll
        for (int t = 0; t < G; ++t)
            acc[t][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w[t]),
                                                                __builtin_bit_cast(bf16x8, x[0]),
                                                                acc[t][0], 0, 0, 0);
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int t = 0; t < G; ++t)
#pragma unroll
                for (int g = 0; g < NX; ++g) {
                    floatx4 &a = acc[G == 1 ? e % 2 : t][g];
                    a = __builtin_amdgcn_mfma_f32_4x4x1f32(__builtin_bit_cast(floatx4, x[g])[e],
                                                           __builtin_bit_cast(floatx4, w[t])[e], a, 0,
                                                           0, 0);
                }
    }
}

// Sum over the four kq of a lane's four envs, one env to each quarter: lane
// l returns output l % 16 of env l / 16.
__device__ __forceinline__ float sum_kq(const floatx4 &a)
{
    typedef unsigned u2 __attribute__((ext_vector_type(2)));
    auto swap32 = [](float x, float y) {   // {x low, y low} + {x high, y high}
        const u2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
        return __uint_as_float(r[0]) + __uint_as_float(r[1]);
    };
    const float p = swap32(a[0], a[2]), q = swap32(a[1], a[3]);
    const u2 r = __builtin_amdgcn_permlane16_swap(__float_as_uint(p), __float_as_uint(q), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// ---------------------------------------------------------------------------
// Matrix role.  NG groups of four envs.  Wave w takes tiles of the hidden
// layers in groups of GT, group i at (i MW + w) GT; layer 1 has at most TW
// groups a wave.
// ---------------------------------------------------------------------------
template <bool BF, int NG, int GT, int TW>
__device__ __forceinline__ void matrix_role(const RolloutArgs &A, const Plan &P, uint8_t *smem,
                                            const uint8_t *pk, int w, int lane)
{
    typedef typename Elem<BF>::T E;
    constexpr int MB = 4 * NG, RU = keep_blocks(GT, NG, TW), NX = XS<BF, NG>;
    const float *bias = (const float *)(smem + P.BIAS);
    u4v ring[16], keep[RU * GT];
    const int lo = lane * 16;
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
        (void *)pk, (short)0, (int)A.lay.agent_stride, 0x00020000);

    // G tiles of a part from tile t0 on (past the last: the last again).
    // Everything derived from a job is the same in every step; computed
    // ahead of the step loop, all of it would need more registers than there
    // are.  Hiding the job from the optimiser at every use keeps it next to
    // its use.
    struct Job {
        int off, kb, KB, first, cut, skip, res, lds, nt, t0;
    };
    auto job = [&](const Part &q, int t0) {
        return Job{q.off, q.kb, q.KB, q.first, q.cut, q.skip, q.res, q.lds, q.nt, t0};
    };
    auto hide = [](Job &j) {
        asm volatile("" : "+s"(j.off), "+s"(j.kb), "+s"(j.KB), "+s"(j.res), "+s"(j.lds), "+s"(j.nt), "+s"(j.t0));
        asm volatile("" : "+s"(j.first), "+s"(j.cut), "+s"(j.skip));
    };
    auto layer_block = [](const Job &j, int k) { return j.first + k + (k >= j.cut ? j.skip : 0); };
    auto gload = [&](const Job &j, int t, int k) {
        return __builtin_bit_cast(u4v, __builtin_amdgcn_raw_buffer_load_b128(
            rsrc, lo, j.off + (min(j.t0 + t, j.nt - 1) * j.KB + layer_block(j, k)) * 1024, 0));
    };
    // the first streamed blocks [res, end)
    auto prime = [&](auto gc, Job j, int end) {
        constexpr int G = decltype(gc)::value, D = flight(G);
        hide(j);
        asm volatile("" : "+s"(end));
#pragma unroll
        for (int d = 0; d < D; ++d)
            if (j.res + d < end)
#pragma unroll
                for (int t = 0; t < G; ++t) ring[d * G + t] = gload(j, t, j.res + d);
    };
    // acc += blocks [0, end): those in LDS, then the streamed ones (primed)
    auto run = [&](auto gc, Job j, int end, const uint8_t *xa, int pitch, auto &acc) {
        constexpr int G = decltype(gc)::value, D = flight(G);
        hide(j);
        asm volatile("" : "+s"(end));
        auto inputs = [&](u4v *x, int k) {
#pragma unroll
            for (int g = 0; g < NX; ++g) x[g] = *(const u4v *)(xa + g * 4 * pitch + layer_block(j, k) * 64);
        };
        if (j.res > 0) {   // two blocks in turn, the next read while one is multiplied
            u4v t[2][G], x[2][NX];
            auto read = [&](int b, int k) {
                k = min(k, j.res - 1);
#pragma unroll
                for (int i = 0; i < G; ++i)
                    t[b][i] = *(const u4v *)(smem + j.lds + (min(j.t0 + i, j.nt - 1) * j.res + k) * 1024 + lo);
                inputs(x[b], k);
            };
            read(0, 0);
            int k = 0;
            for (; k + 2 <= j.res; k += 2) {
                read(1, k + 1);
                block<BF, NX, G>(t[0], x[0], acc);
                read(0, k + 2);
                block<BF, NX, G>(t[1], x[1], acc);
            }
            if (k < j.res) block<BF, NX, G>(t[0], x[0], acc);
        }
        int k = j.res;
        if (k >= end) return;
        u4v x[2][NX];
        inputs(x[0], k);
        for (; k + D <= end; k += D)
#pragma unroll
            for (int d = 0; d < D; ++d) {
                inputs(x[(d + 1) & 1], min(k + d + 1, end - 1));
                block<BF, NX, G>(ring + d * G, x[d & 1], acc);
                const int next = min(k + d + D, end - 1);
#pragma unroll
                for (int t = 0; t < G; ++t) ring[d * G + t] = gload(j, t, next);
                __builtin_amdgcn_sched_barrier(0);   // the refill stays here
            }
#pragma unroll
        for (int d = 0; d < D - 1; ++d)
            if (k + d < end) {
                inputs(x[(d + 1) & 1], min(k + d + 1, end - 1));
                block<BF, NX, G>(ring + d * G, x[d & 1], acc);
            }
    };
    // inputs kq = lane / 16 of env lane % 4 (bf16: lane % MB)
    const int xl = (lane / 16) * 16, xe = lane % (BF ? MB : 4);
    const uint8_t *x0 = smem + P.X + xe * P.ldx + xl;
    const uint8_t *h1 = smem + P.H1 + xe * P.ldh1 + xl;
    const uint8_t *h2 = smem + P.H2 + xe * P.ldh2 + xl;
    // finish G tiles of layer l from t0 on.  A lane takes NG (output, env) pairs
    // of a tile: fp32 output lane % 16 of envs lane / 16 + 4 g, bf16 output
    // 4 (lane / 16) + lane % 16 / MB NG + g of env lane % MB.  Nothing is
    // conditional, so the tiles' chains interleave: a tile past the last repeats
    // the last one's values, and outputs past the layer's have room in their
    // rows: zeros, not what their zero weights give, which is NaN where an
    // input is infinite.
    auto finish = [&](auto lc, auto gc, const Part &q, int t0, const auto &acc) {
        constexpr int l = decltype(lc)::value, G = decltype(gc)::value;
        const float *b = bias + (l == 0 ? 0 : l == 1 ? P.part[0].nt : P.part[0].nt + P.part[2].nt) * 16;
        const int sub = lane % 16 / MB;   // bf16: which NG of a lane's outputs it takes
        int o[G];
        float v[G][NG];
#pragma unroll
        for (int t = 0; t < G; ++t) {
            o[t] = min(t0 + t, q.nt - 1) * 16 + (BF ? lane / 16 * 4 + sub * NG : lane % 16);
            if constexpr (BF) {
                // register sub NG + g, by compares (MB = 16: sub is 0)
                const floatx4 &a = acc[t][0];
#pragma unroll
                for (int g = 0; g < NG; ++g) {
                    float x = a[g];
#pragma unroll
                    for (int i = 1; i < 4 / NG; ++i) x = sub == i ? a[i * NG + g] : x;
                    v[t][g] = x + b[o[t] + g];
                }
            } else {
                const float bo = b[o[t]];
#pragma unroll
                for (int g = 0; g < NG; ++g)
                    v[t][g] = sum_kq(G == 1 ? acc[0][g] + acc[ACCS<BF, G> - 1][g] : acc[t][g]) + bo;
            }
        }
        if constexpr (l < 2) {
#pragma unroll
            for (int t = 0; t < G; ++t)
#pragma unroll
                for (int g = 0; g < NG; ++g) {
                    const float h = BF ? tanh_for_bf16(v[t][g]) : tanh_f32(v[t][g]);
                    v[t][g] = BF || o[t] < q.out ? h : 0.f;   // (bf16 widths are whole tiles)
                }
        }
#pragma unroll
        for (int t = 0; t < G; ++t)
#pragma unroll
            for (int g = 0; g < NG; ++g) {
                const int m = BF ? lane % MB : g * 4 + lane / 16, c = o[t] + (BF ? g : 0);
                if constexpr (l == 2) ((float *)(smem + P.MU))[m * P.ldm + c] = v[t][g];
                else ((E *)(smem + (l == 0 ? P.H1 + m * P.ldh1 : P.H2 + m * P.ldh2)))[c] = cvt<BF>(v[t][g]);
            }
    };
    auto clear = [&](auto &acc) {
        for (auto &r : acc)
            for (auto &v : r) v = floatx4{0.f, 0.f, 0.f, 0.f};
    };

    const ic<GT> g;
    const int t0 = w * GT;                                    // this wave's first group
    const Job jm = job(P.part[0], t0), ja = job(P.part[1], t0), j2 = job(P.part[2], t0);
    const Job j3 = job(P.part[3], w);
    const bool has1 = t0 < jm.nt, has2 = t0 < j2.nt, has3 = w < j3.nt;
    // the ring is free through slot B where no state column streams in one
    // group, from layer 2's last streamed block to slot A where layer 3 does not
    const bool earlyB = TW == 1 && ja.res == ja.kb;
    const bool earlyA = j2.nt <= MW * GT && j3.res == j3.kb;
    const int k2 = max(j2.res, j2.kb - RU);   // layer 2's blocks from here on are in `keep`
    if (has2)
#pragma unroll
        for (int d = 0; d < RU; ++d)
            if (k2 + d < j2.kb)
#pragma unroll
                for (int t = 0; t < GT; ++t) keep[d * GT + t] = gload(j2, t, k2 + d);
    if (has1) prime(g, jm, jm.kb);
    __syncthreads();   // rows, biases and resident weights are in LDS
    for (int j = 0; j < A.L; ++j) {
        const uint8_t *x = x0 + (j & 1) * (MB * P.ldx);
        // slot A: market columns of layer 1
        floatx4 z[TW][ACCS<BF, GT>][NX];
#pragma unroll
        for (int i = 0; i < TW; ++i) {
            clear(z[i]);
            const Job q = job(P.part[0], (i * MW + w) * GT);
            if (q.t0 < q.nt) {
                if (i > 0) prime(g, q, q.kb);
                run(g, q, q.kb, x, P.ldx, z[i]);
            }
        }
        if (has1) prime(g, ja, ja.kb);
        __syncthreads();
        // slot B: state columns, h1 (the next streamed blocks go out as soon as
        // the ring is free)
        if (earlyB && has2) prime(g, j2, k2);
#pragma unroll
        for (int i = 0; i < TW; ++i) {
            const Job q = job(P.part[1], (i * MW + w) * GT);
            if (q.t0 < q.nt) {
                if (i > 0) prime(g, q, q.kb);
                run(g, q, q.kb, x, P.ldx, z[i]);
                finish(ic<0>{}, g, P.part[0], q.t0, z[i]);
            }
        }
        if (!earlyB && has2) prime(g, j2, k2);
        __syncthreads();
        // slot L2: the first group with its registers, the others streamed
        if (has2) {
            floatx4 acc[ACCS<BF, GT>][NX];
            clear(acc);
            run(g, j2, k2, h1, P.ldh1, acc);
            if (earlyA && has1) prime(g, jm, jm.kb);
            int k = k2, n = j2.kb - k2;
            asm volatile("" : "+s"(k), "+s"(n));
            u4v x[2][NX];
            auto inputs = [&](int b, int d) {
#pragma unroll
                for (int i = 0; i < NX; ++i)
                    x[b][i] = *(const u4v *)(h1 + i * 4 * P.ldh1 + (k + min(d, n - 1)) * 64);
            };
            inputs(0, 0);
#pragma unroll
            for (int d = 0; d < RU; ++d)
                if (d < n) {
                    if (d + 1 < RU) inputs((d + 1) & 1, d + 1);
                    block<BF, NX, GT>(keep + d * GT, x[d & 1], acc);
                }
            finish(ic<1>{}, g, P.part[2], t0, acc);
        }
        for (int t = t0 + MW * GT; t < P.part[2].nt; t += MW * GT) {
            const Job q = job(P.part[2], t);
            floatx4 acc[ACCS<BF, GT>][NX];
            clear(acc);
            prime(g, q, q.kb);
            run(g, q, q.kb, h1, P.ldh1, acc);
            finish(ic<1>{}, g, P.part[2], t, acc);
        }
        if (earlyA && has1 && !has2) prime(g, jm, jm.kb);
        if (has3) prime(ic<1>{}, j3, j3.kb);
        __syncthreads();
        // slot L3 (at most two tiles a wave)
        for (int t = w; t < P.part[3].nt; t += MW) {
            const Job q = job(P.part[3], t);
            floatx4 acc[ACCS<BF, 1>][NX];
            clear(acc);
            if (t != w) prime(ic<1>{}, q, q.kb);
            run(ic<1>{}, q, q.kb, h2, P.ldh2, acc);
            finish(ic<2>{}, ic<1>{}, P.part[3], t, acc);
        }
        if (!earlyA && has1) prime(g, jm, jm.kb);
        __syncthreads();
    }
    __syncthreads();   // the last env step
}

// ---------------------------------------------------------------------------
// Env roles: wave v of each kind owns env slots 4 v .. 4 v + 3
// ---------------------------------------------------------------------------
struct Slot {
    int sl, e, agent;     // slot in the workgroup, env, agent
    bool mine, live;      // the slot holds an env; it is stepped
    int64_t t0;
};

__device__ __forceinline__ Slot env_slot(const RolloutArgs &A, int agent, int ebase, int nenv, int v,
                                         int lane)
{
    Slot s;
    s.sl = 4 * v + lane / RL;
    s.mine = s.sl < nenv;
    s.e = ebase + s.sl;
    s.agent = agent;
    s.t0 = s.mine ? A.t[s.e] : -1;
    s.live = s.t0 >= 0 && s.t0 <= A.env.T1 - 1 - A.L;
    return s;
}

template <bool BF, int N>
__device__ __forceinline__ void trade_role(const RolloutArgs &A, const Plan &P, uint8_t *smem,
                                           const Slot s, int MB, int lane)
{
    typedef typename Elem<BF>::T E;
    const EnvConst &C = A.env;
    const int n = C.n, sl16 = lane % RL, i0 = N * sl16;
    const size_t EE = (size_t)A.E;
    const float qnan = __builtin_nanf("");   // (taps of envs not stepped)
    if (A.n_invalid && s.mine && !s.live && sl16 == 0) atomicAdd(A.n_invalid, 1);

    // the trade is the longest part of the chain: it goes first on its SIMD
    __builtin_amdgcn_s_setprio(3);
    RowEnvN<N> st;
    st.cash = s.mine ? A.cash[s.e] : 0.0;
    double hv = 0.0;
#pragma unroll
    for (int c = 0; c < N; ++c) {
        const bool in = s.mine && i0 + c < n;
        st.h[c] = in ? A.shares[(size_t)s.e * n + i0 + c] : 0;
        st.pd[c] = in && s.live ? (double)C.price[(size_t)s.t0 * n + i0 + c] : 0.0;
        hv = fma((double)st.h[c], st.pd[c], hv);
    }
    st.value = st.cash + row_sum(hv);
    const bool wave_live = __ballot(s.live) != 0;

    // the balance and the holdings of the row in buffer b
    auto write_state = [&](int b) {
        if (!s.live) return;
        E *x = (E *)(smem + P.X + (b * MB + s.sl) * P.ldx);
        if (sl16 == 0) x[0] = cvt<BF>((float)(st.cash * (double)C.cash_scale));
#pragma unroll
        for (int c = 0; c < N; ++c)
            if (i0 + c < n) x[1 + n + i0 + c] = cvt<BF>((float)st.h[c] * C.share_scale);
    };
    write_state(0);
    __syncthreads();

    // env step j (mu, normals and next prices are in LDS).  It touches no
    // global memory but for taps: a store would queue behind the weight loads.
    auto step = [&](int j) {
        const int pj = (j & 1) * MB + s.sl, pn = ((j + 1) & 1) * MB + s.sl;
        const float *mu = (const float *)(smem + P.MU) + s.sl * P.ldm + i0;
        const float *sz = (const float *)(smem + P.SZ) + pj * P.ldm + i0;
        const float *nx = (const float *)(smem + P.PN) + pn * P.ldm + i0;
        float a[N];
        double qd[N];
#pragma unroll
        for (int c = 0; c < N; ++c) {
            const bool in = s.live && i0 + c < n;
            a[c] = in ? mu[c] + sz[c] : 0.f;
            qd[c] = in ? (double)nx[c] : 0.0;
        }
        float rw = 0.f;
        if (wave_live) rw = env_step_row(C, st, a, qd);
        write_state((j + 1) & 1);
        if (sl16 == 0) ((float *)(smem + P.RW))[s.sl] = rw;
        if (!s.mine) return;
        const size_t row = (size_t)j * EE + s.e;
        if (A.shares_tap) {
#pragma unroll
            for (int c = 0; c < N; ++c)
                if (i0 + c < n) A.shares_tap[row * n + i0 + c] = st.h[c];
        }
        if (sl16 == 0) {
            if (A.cash_tap) A.cash_tap[row] = st.cash;
            if (A.asset_tap) A.asset_tap[row] = s.live ? st.value : (double)qnan;
        }
    };
    for (int j = 0; j < A.L; ++j) {
        if (j > 0) step(j - 1);
        for (int i = 0; i < 4; ++i) __syncthreads();
    }
    step(A.L - 1);
    __syncthreads();
    if (s.live) {
        if (sl16 == 0) {
            A.cash[s.e] = st.cash;
            A.t[s.e] = s.t0 + A.L;
        }
#pragma unroll
        for (int c = 0; c < N; ++c)
            if (i0 + c < n) A.shares[(size_t)s.e * n + i0 + c] = st.h[c];
    }
}

template <bool BF>
__device__ __forceinline__ void aux_role(const RolloutArgs &A, const Plan &P, uint8_t *smem,
                                         const uint8_t *pk, const Slot s, int MB, int lane)
{
    typedef typename Elem<BF>::T E;
    __builtin_amdgcn_s_setprio(2);   // ahead of the matrix wave of its SIMD
    constexpr int VE = 16 / (int)sizeof(E);
    constexpr int NQ = 2;    // Philox counters a lane takes (4 stocks each)
    constexpr int NM = 16;   // indicators a lane has in flight
    const EnvConst &C = A.env;
    const int n = C.n, sl16 = lane % RL;
    const size_t EE = (size_t)A.E;
    const float qnan = __builtin_nanf("");

    // market row t0 + d: prices sl16 + 16 m, indicators sl16 + 16 (m0 + m).
    // (The lane's index and the counts are hidden from the optimiser, which
    // would keep every index and mask in registers through the step loop.)
    float pv[8], iv[NM];
    auto load_ind = [&](int d, int m0) {
        int i0 = sl16, nI = C.nI;
        asm volatile("" : "+v"(i0), "+s"(nI));
        const float *ir = C.ind + (size_t)(s.live ? s.t0 + d : 0) * nI;
#pragma unroll
        for (int m = 0; m < NM; ++m) {
            if (RL * (m0 + m) >= nI) break;
            iv[m] = __builtin_nontemporal_load(ir + min(i0 + RL * (m0 + m), nI - 1));
        }
    };
    auto load = [&](int d) {
        int i0 = sl16, n = C.n;
        asm volatile("" : "+v"(i0), "+s"(n));
        const float *pr = C.price + (size_t)(s.live ? s.t0 + d : 0) * n;
#pragma unroll
        for (int m = 0; m < 8; ++m) {
            if (RL * m >= n) break;
            pv[m] = __builtin_nontemporal_load(pr + min(i0 + RL * m, n - 1));
        }
        load_ind(d, 0);
    };
    // ... into the rows of step d, and the next prices
    auto put_ind = [&](int d, int m0) {
        int i0 = sl16, nI = s.live ? C.nI : 0, all = C.nI;
        asm volatile("" : "+v"(i0), "+v"(nI), "+s"(all));
        E *x = (E *)(smem + P.X + ((d & 1) * MB + s.sl) * P.ldx) + 1 + 2 * n;
#pragma unroll
        for (int m = 0; m < NM; ++m) {
            if (RL * (m0 + m) >= all) break;
            const int i = i0 + RL * (m0 + m);
            if (i < nI) x[i] = cvt<BF>(iv[m]);
        }
    };
    auto write_market = [&](int d) {
        {
            int i0 = sl16, np = s.live ? n : 0, all = n;
            asm volatile("" : "+v"(i0), "+v"(np), "+s"(all));
            E *x = (E *)(smem + P.X + ((d & 1) * MB + s.sl) * P.ldx) + 1;
            float *pn = (float *)(smem + P.PN) + ((d & 1) * MB + s.sl) * P.ldm;
#pragma unroll
            for (int m = 0; m < 8; ++m) {
                if (RL * m >= all) break;
                const int i = i0 + RL * m;
                if (i < np) {
                    x[i] = cvt<BF>(pv[m] * C.price_scale);
                    pn[i] = pv[m];
                }
            }
        }
        put_ind(d, 0);
        for (int m0 = NM; RL * m0 < C.nI; m0 += NM) {
            load_ind(d, m0);
            put_ind(d, m0);
        }
    };
    // the observation row in buffer b
    auto store_obs = [&](int b, E *dst) {
        const u4v *x = (const u4v *)(smem + P.X + (b * MB + s.sl) * P.ldx);
#pragma unroll 4
        for (int c = sl16; c < C.K_pad / VE; c += RL) __builtin_nontemporal_store(x[c], (u4v *)dst + c);
    };
    float ls[NQ][4], sg[NQ][4];
    const float *lsd = (const float *)(pk + A.lay.off_ls);
#pragma unroll
    for (int q = 0; q < NQ; ++q)
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int i = 4 * (sl16 + RL * q) + c;
            ls[q][c] = i < n ? lsd[i] : 0.f;
            sg[q][c] = expf(ls[q][c]);
        }
    const double half_log2pi_n = 0.5 * (double)n * 1.8378770664093454836;
    // normals of step j (times sigma) and their log-density
    auto normals = [&](int j) {
        const int pj = (j & 1) * MB + s.sl;
        float *sz = (float *)(smem + P.SZ) + pj * P.ldm;
        double l = 0.0;
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const int k = sl16 + RL * q;
            if (4 * RL * q >= n) break;
            const U4 w = philox4x32_10(U4{(uint32_t)k, (uint32_t)s.e, (uint32_t)(A.step0 + (uint64_t)j),
                                          (uint32_t)s.agent},
                                       A.key_lo, A.key_hi);
            float z[4];
            box_muller(uniform_open01(w.x), uniform_open01(w.y), z[0], z[1]);
            box_muller(uniform_open01(w.z), uniform_open01(w.w), z[2], z[3]);
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (4 * k + c < n) {
                    sz[4 * k + c] = sg[q][c] * z[c];
                    l += -0.5 * (double)z[c] * (double)z[c] - (double)ls[q][c];
                }
        }
        l = row_sum(l) - half_log2pi_n;
        if (sl16 == 0) ((double *)(smem + P.LP))[pj] = l;
    };
    // the trajectory row of step j, after its env step
    auto store_row = [&](int j) {
        if (!s.mine) return;
        const size_t row = (size_t)j * EE + s.e;
        const int pj = (j & 1) * MB + s.sl;
        const float *mu = (const float *)(smem + P.MU) + s.sl * P.ldm;
        const float *sz = (const float *)(smem + P.SZ) + pj * P.ldm;
        for (int i = sl16; i < n; i += RL) {
            const float m = mu[i];
            __builtin_nontemporal_store(s.live ? m + sz[i] : qnan, A.action + row * n + i);
            if (A.mu_tap) __builtin_nontemporal_store(s.live ? m : qnan, A.mu_tap + row * n + i);
        }
        if (sl16 == 0) {
            const bool done = A.step0 + (uint64_t)j + 1 == (uint64_t)C.horizon;
            A.logp[row] = s.live ? (float)((const double *)(smem + P.LP))[pj] : qnan;
            A.reward[row] = s.live ? ((const float *)(smem + P.RW))[s.sl] : qnan;
            A.done[row] = s.live ? (uint8_t)done : (uint8_t)0;
        }
    };

    load(0);
    write_market(0);
    load(1);
    __syncthreads();
    for (int j = 0; j < A.L; ++j) {
        // slot A
        normals(j);
        write_market(j + 1);
        __syncthreads();
        // slot B
        __syncthreads();
        // slot L2
        if (j > 0) store_row(j - 1);
        __syncthreads();
        // slot L3: stores before the loads, which the next slot A waits for
        if (A.obs && s.live) store_obs(j & 1, (E *)A.obs + ((size_t)j * EE + s.e) * A.ld_obs);
        if (j + 2 <= A.L) load(j + 2);
        __syncthreads();
    }
    __syncthreads();
    store_row(A.L - 1);
    if (A.obs_last && s.live) store_obs(A.L & 1, (E *)A.obs_last + (size_t)s.e * A.ld_obs);
}

template <bool BF, int NG, int GT, int TW, int N>
__global__ __launch_bounds__((MW + 2 * NG) * WAVE) void rollout_four_kernel(RolloutArgs A, Plan P)
{
    constexpr int MB = 4 * NG, NTH = (MW + 2 * NG) * WAVE;
    extern __shared__ __align__(16) uint8_t smem[];
    const int tid = threadIdx.x, lane = tid % WAVE;
    const int wave = __builtin_amdgcn_readfirstlane(tid / WAVE);
    // XCD-aware block order: an agent's blocks share an XCD and its L2
    const int nb = gridDim.x;
    const int logical = (blockIdx.x % 8) * (nb / 8) + blockIdx.x / 8;
    if (logical >= A.n_agents * A.blocks_per_agent) return;
    const int agent = logical / A.blocks_per_agent, blk = logical % A.blocks_per_agent;
    const int ebase = agent * A.envs_per_agent + blk * MB;
    const int nenv = min(MB, A.envs_per_agent - blk * MB);
    const uint8_t *pk = A.packed + (size_t)agent * A.lay.agent_stride;

    // rows and hidden rows zero (padding and absent envs stay so), biases
    // and resident weights
    for (int i = tid; i < P.MU / 16; i += NTH) ((u4v *)smem)[i] = u4v{0, 0, 0, 0};
    float *bias = (float *)(smem + P.BIAS);
    int at = 0;
    for (int l = 0; l < 3; ++l) {
        const Part &q = P.part[l == 0 ? 0 : l + 1];
        const float *src = (const float *)(pk + A.lay.off_b[l]);
        for (int i = tid; i < q.nt * 16; i += NTH) bias[at + i] = i < q.out ? src[i] : 0.f;
        at += q.nt * 16;
    }
    for (int p = 0; p < 4; ++p) {
        const Part &q = P.part[p];
        for (int b = wave; b < q.nt * q.res; b += NTH / WAVE) {
            const int k = b % q.res, kk = q.first + k + (k >= q.cut ? q.skip : 0);
            ((u4v *)(smem + q.lds))[b * WAVE + lane] =
                ((const u4v *)(pk + q.off))[(b / q.res * q.KB + kk) * WAVE + lane];
        }
    }
    __syncthreads();

    if (wave < MW) {
        matrix_role<BF, NG, GT, TW>(A, P, smem, pk, wave, lane);
    } else {
        const Slot s = env_slot(A, agent, ebase, nenv, (wave - MW) / 2, lane);
        if ((wave - MW) % 2 == 0)
            trade_role<BF, N>(A, P, smem, s, MB, lane);
        else
            aux_role<BF>(A, P, smem, pk, s, MB, lane);
    }
}

// ---------------------------------------------------------------------------
// Launch
// ---------------------------------------------------------------------------
// pitch of rows of `bytes`: 64 past a multiple of 256, so that the four
// envs' 64 bytes of a k-block fall on different banks
inline int pitch(int bytes) { return (bytes - 64 + 255) / 256 * 256 + 64; }

inline bool make_plan(const PackedLayout &L, int MB, int GT, int TW, int budget, Plan *P)
{
    const int es = L.dtype == TP_BF16 ? 2 : 4, per = 64 / es;
    const int n = L.n, S = L.S;
    auto blocks = [&](int k) { return (k + per - 1) / per; };
    // layer 1's state blocks: block 0 (the balance) and b0 .. b1 (the
    // holdings, columns n + 1 .. 2n)
    const int all = blocks(S), b1 = 2 * n / per, b0 = (n + 1) / per > 1 ? (n + 1) / per : 1;
    const int held = b1 >= b0 ? b1 - b0 + 1 : 0;
    const int u2 = blocks(L.H1), u3 = blocks(L.H2);
    const int outs[4] = {L.H1, L.H1, L.H2, L.n}, kbs[4] = {all - 1 - held, 1 + held, u2, u3};
    for (int p = 0; p < 4; ++p) {
        Part &q = P->part[p];
        q.out = outs[p];
        q.nt = (q.out + 15) / 16;
        q.kb = kbs[p];
        q.KB = L.KS[p < 2 ? 0 : p - 1];
        q.first = p == 0 ? 1 : 0;
        q.cut = p == 0 ? b0 - 1 : p == 1 ? 1 : 1 << 30;
        q.skip = p == 0 ? held : p == 1 ? b0 - 1 : 0;
        q.off = (int)L.off_W[p < 2 ? 0 : p - 1];
    }
    const int N = n <= 32 ? 2 : 8;
    P->ldm = RL * N;
    P->ldx = pitch(blocks(L.K_pad) * 64);
    P->ldh1 = pitch(u2 * 64);
    P->ldh2 = pitch(u3 * 64);
    int o = 0;
    auto area = [&](int bytes) {
        const int r = o;
        o = (o + bytes + 15) & ~15;
        return r;
    };
    P->X = area(2 * MB * P->ldx);
    P->H1 = area(MB * P->ldh1);
    P->H2 = area(MB * P->ldh2);
    P->MU = area(MB * P->ldm * 4);
    P->SZ = area(2 * MB * P->ldm * 4);
    P->PN = area(2 * MB * P->ldm * 4);
    P->LP = area(2 * MB * 8);
    P->RW = area(MB * 4);
    P->BIAS = area((P->part[0].nt + P->part[2].nt + P->part[3].nt) * 64);
    if (o > budget) return false;
    // resident weights, whole k-blocks of every tile: the action layer, the
    // state columns, layer 2 (but for what the matrix waves keep in
    // registers), the market columns
    const int keep = keep_blocks(GT, MB / 4, TW);
    for (int p : {3, 1, 2, 0}) {
        Part &q = P->part[p];
        int want = q.kb;
        if (p == 2 && q.nt <= MW * GT) want = want > keep ? want - keep : 0;
        const int fit = (budget - o) / (q.nt * 1024);
        q.res = fit < want ? fit : want;
        q.lds = area(q.res * q.nt * 1024);
    }
    P->bytes = o;
    return true;
}

template <bool BF, int NG, int GT, int TW, int N>
hipError_t launch_cfg(RolloutArgs &a, const Plan &P, hipStream_t s)
{
    auto k = rollout_four_kernel<BF, NG, GT, TW, N>;
    const hipError_t e = hipFuncSetAttribute((const void *)k,
                                             hipFuncAttributeMaxDynamicSharedMemorySize, P.bytes);
    if (e != hipSuccess) return e;
    a.blocks_per_agent = (a.envs_per_agent + 4 * NG - 1) / (4 * NG);
    const int nblk = (a.n_agents * a.blocks_per_agent + 7) & ~7;
    hipLaunchKernelGGL(k, dim3(nblk), dim3((MW + 2 * NG) * WAVE), P.bytes, s, a, P);
    return hipGetLastError();
}

// The hidden widths' tile groups
struct Tiles {
    int GT, TW;
};
inline Tiles tiles(const PackedLayout &L)
{
    const int H = L.H1 > L.H2 ? L.H1 : L.H2, nt1 = (L.H1 + 15) / 16;
    const int GT = H <= 64 ? 1 : H <= 128 ? 2 : nt1 > 4 * MW && nt1 <= 6 * MW ? 3 : 4;
    return {GT, nt1 <= GT * MW ? 1 : GT == 3 ? 2 : 4};
}

// NG env groups of four
template <bool BF, int NG, int N>
hipError_t launch_width(RolloutArgs &a, hipStream_t s)
{
    const Tiles t = tiles(a.lay);
    Plan P;
    if (!make_plan(a.lay, 4 * NG, t.GT, t.TW, (int)LDS_LIMIT, &P)) return hipErrorNotSupported;
    if (t.GT == 2) return launch_cfg<BF, NG, 2, 1, N>(a, P, s);
    if (t.GT == 3) return launch_cfg<BF, NG, 3, 2, N>(a, P, s);
    if constexpr (!BF) {   // (bf16 widths are multiples of 128, first layers at most 384 wide)
        if (t.GT == 1) return launch_cfg<BF, NG, 1, 1, N>(a, P, s);
        if (t.TW == 4) return launch_cfg<BF, NG, 4, 4, N>(a, P, s);
    }
    return launch_cfg<BF, NG, 4, 1, N>(a, P, s);
}

template <bool BF, int N>
hipError_t launch_type(RolloutArgs &a, hipStream_t s)
{
    auto blocks = [&](int MB) { return (int64_t)a.n_agents * ((a.envs_per_agent + MB - 1) / MB); };
    if constexpr (BF)   // (every bf16 shape taken fits 16 envs)
        if (blocks(8) > 256) return launch_width<BF, 4, N>(a, s);
    if (blocks(4) > 256) {
        const hipError_t e = launch_width<BF, 2, N>(a, s);
        if (e != hipErrorNotSupported) return e;
    }
    return launch_width<BF, 1, N>(a, s);
}

}  // namespace four
}  // namespace tpk
