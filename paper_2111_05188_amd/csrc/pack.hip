// Parameter packing: fp32 masters -> the rollout and critic kernels' layouts,
// one launch for all matrices and vectors of all agents. Separate launches take
// about 4.5 us each on a busy queue, whatever their size: a generation of 16
// pods of a 100-stock 512-wide bf16 network (critic and actor) spent 0.65 ms of
// its 12.5 ms on 208 of them; the two launches now take 28 us each, nearly all
// of it the 63 MB of fp32 masters that they read.
#include "device.hpp"
#include "internal.hpp"

namespace tpk {

namespace {

enum PackKind : int {
    // MFMA A-fragments [NT][KB][64 lanes][16 bytes], zero outside [out][in]:
    PACK_FRAG_BF16,   // lane l, element e: W[16t + l%16][32b + 8(l/16) + e]
    PACK_FRAG_F32,    // W[16t + l%16][16b + 4(l/16) + e]
    PACK_KBLOCK,      // [KB][out][4]: W[o][4 b + e], zero for inputs past `in`
    PACK_VEC,         // out values, zeros to the last piece
    PACK_VEC_BF16,    // the same, rounded to bf16 (kept in fp32 storage)
};

// One matrix or vector of an agent: `pieces` 16-byte pieces at dst_off of
// the agent's packed parameters, from src + agent * src_stride floats.
struct PackSeg {
    const float *src;
    int64_t src_stride;
    size_t dst_off;
    int kind, out, in, NT, KB;
    int pieces, block0;   // first workgroup of this segment
};
constexpr int MAX_PACK = 7;
constexpr int PT = 256;   // threads (and pieces) per workgroup
struct PackBatch {
    PackSeg s[MAX_PACK];
    int n, blocks;
    uint8_t *dst;
    size_t dst_stride;
};

__global__ __launch_bounds__(PT) void pack_kernel(PackBatch pb)
{
    int si = 0;
#pragma unroll
    for (int q = 1; q < MAX_PACK; ++q)
        if (q < pb.n && (int)blockIdx.x >= pb.s[q].block0) si = q;
    const PackSeg S = pb.s[si];
    const int p = ((int)blockIdx.x - S.block0) * PT + (int)threadIdx.x;
    if (p >= S.pieces) return;
    const float *W = S.src + (size_t)blockIdx.y * S.src_stride;
    uint8_t *dst = pb.dst + blockIdx.y * pb.dst_stride + S.dst_off + (size_t)p * 16;
    if (S.kind == PACK_VEC || S.kind == PACK_VEC_BF16) {
        floatx4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float x = 4 * p + e < S.out ? W[4 * p + e] : 0.0f;
            v[e] = S.kind == PACK_VEC ? x : (float)to_bf16(x);
        }
        *(floatx4 *)dst = v;
        return;
    }
    int o, k, step = 4;
    if (S.kind == PACK_KBLOCK) {
        o = p % S.out;
        k = p / S.out * 4;
    } else {
        step = S.kind == PACK_FRAG_BF16 ? 8 : 4;
        const int lane = p % WAVE, b = p / WAVE % S.KB, t = p / WAVE / S.KB;
        o = 16 * t + lane % 16;
        k = step * (4 * b + lane / 16);
    }
    const float *row = W + (size_t)o * S.in;
    float x[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = e < step && o < S.out && k + e < S.in ? row[k + e] : 0.0f;
    if (S.kind == PACK_FRAG_BF16) {
        bf16x8 v;
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = to_bf16(x[e]);
        *(bf16x8 *)dst = v;
    } else {
        *(floatx4 *)dst = floatx4{x[0], x[1], x[2], x[3]};
    }
}

struct Packer {
    PackBatch b{};
    // `stride`: floats between agents in this array
    void add(int kind, const float *src, int64_t stride, size_t off, int out, int in, int NT, int KB,
             int64_t pieces)
    {
        PackSeg &s = b.s[b.n++];
        s = PackSeg{src, stride, off, kind, out, in, NT, KB, (int)pieces, b.blocks};
        b.blocks += (int)((pieces + PT - 1) / PT);
    }
    void frag(int dtype, const float *W, int64_t stride, size_t off, int out, int in, int NT, int KB)
    {
        add(dtype == TP_BF16 ? PACK_FRAG_BF16 : PACK_FRAG_F32, W, stride, off, out, in, NT, KB,
            (int64_t)NT * KB * WAVE);
    }
    // cnt values, zeros up to `padded` (whole pieces: the areas are 256-byte
    // aligned, so the last piece's end is the layout's own padding)
    void vec(bool round, const float *src, int64_t stride, size_t off, int cnt, int padded)
    {
        add(round ? PACK_VEC_BF16 : PACK_VEC, src, stride, off, cnt, 1, 0, 0, (padded + 3) / 4);
    }
    hipError_t launch(void *dst, size_t dst_stride, int agents, hipStream_t s)
    {
        b.dst = (uint8_t *)dst;
        b.dst_stride = dst_stride;
        for (int a0 = 0; a0 < agents; a0 += 65535) {
            const int n = agents - a0 < 65535 ? agents - a0 : 65535;
            hipLaunchKernelGGL(pack_kernel, dim3(b.blocks, n), dim3(PT), 0, s, b);
            b.dst += (size_t)n * dst_stride;
            for (int i = 0; i < b.n; ++i) b.s[i].src += (size_t)n * b.s[i].src_stride;
        }
        return hipGetLastError();
    }
};

}  // namespace

hipError_t launch_critic_pack(const tp_critic *c, const CriticLayout &L, void *dst, hipStream_t s)
{
    const int outs[2] = {L.H1, L.H2}, ins[2] = {L.S, L.H1};
    auto stride = [&](int64_t own) { return c->agent_stride ? c->agent_stride : own; };
    Packer p;
    for (int l = 0; l < 2; ++l) {
        p.frag(L.dtype, c->W[l], stride((int64_t)outs[l] * ins[l]), L.off_W[l], outs[l], ins[l],
               L.NT[l], L.KS[l]);
        p.vec(false, c->b[l], stride(outs[l]), L.off_b[l], outs[l], 16 * L.NT[l]);
    }
    p.vec(L.dtype == TP_BF16, c->W[2], stride(L.H2), L.off_W[2], L.H2, 16 * L.NT[1]);
    p.vec(false, c->b[2], stride(1), L.off_b[2], 1, 1);
    return p.launch(dst, L.agent_stride, c->n_agents, s);
}

hipError_t launch_pack(const tp_actor *a, const PackedLayout &L, void *dst, hipStream_t s)
{
    const int outs[3] = {L.H1, L.H2, L.n}, ins[3] = {L.S, L.H1, L.H2};
    auto stride = [&](int64_t own) { return a->agent_stride ? a->agent_stride : own; };
    const bool bf = L.dtype == TP_BF16;
    Packer p;
    for (int l = 0; l < 3; ++l) {
        const int64_t st = stride((int64_t)outs[l] * ins[l]);
        if (bf || L.four)
            p.frag(L.dtype, a->W[l], st, L.off_W[l], outs[l], ins[l], L.NT[l], L.KS[l]);
        else
            p.add(PACK_KBLOCK, a->W[l], st, L.off_W[l], outs[l], ins[l], 0, 0,
                  (int64_t)L.KS[l] * outs[l]);
        p.vec(false, a->b[l], stride(outs[l]), L.off_b[l], outs[l], bf ? L.NT[l] * 16 : outs[l]);
    }
    p.vec(false, a->log_std, stride(L.n), L.off_ls, L.n, bf ? L.NT[2] * 16 : L.n);
    return p.launch(dst, L.agent_stride, a->n_agents, s);
}

}  // namespace tpk
