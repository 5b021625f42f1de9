// dlm_block_attn_bwd: gradients of block attention (dQ, and dK / dV per KV segment).
//
// With P = softmax(scale Q K^T + mask), O = P V and an upstream gradient dO:
//   delta_r = sum_c dO[r,c] O[r,c]                  (= rowsum(dP * P))
//   dV = P^T dO,  dP = dO V^T,  dS = P * (dP - delta),  dQ = scale dS K,  dK = scale dS^T Q.
// P is recomputed from Q, K and the forward pass's log-sum-exp; nothing of size Lq x Lk is stored.
//
// No atomics, every output element written exactly once (deterministic):
//   * attn_bwd_delta_kernel : delta per (sequence, head, query row), where the dQ kernel below does not form it.
//   * attn_bwd_dq_kernel    : a workgroup owns 128 rows (query, head in group) of one (sequence, KV head) and
//                             walks the key tiles of all segments, like the forward kernel.  Per 32-key tile and
//                             wavefront: S^T = K Q^T and dP^T = V dO^T (keys are the MFMA rows, so a lane holds 16
//                             keys of ONE query row and LSE / delta are per-lane scalars), dS^T in registers is
//                             already the B operand of dQ^T += K^T dS^T; K^T fragments come from LDS through the
//                             transposing 64-bit LDS read.  attn_bwd_dq64_kernel: the same with 64 rows a wavefront.
//   * attn_bwd_dkv_kernel   : the mirror image.  A workgroup owns 64 or 128 keys of ONE segment of one (sequence, KV
//                             head) and walks the 32-row tiles of (query, head in group) rows that can see them:
//                             S = Q K^T and dP = dO V^T (rows are the MFMA rows, a lane holds 16 rows of ONE key), P
//                             and dS in registers are the B operands of dV^T += dO^T P and dK^T += Q^T dS; the sum
//                             over the heads of a group happens in the accumulators because the rows of all its
//                             heads pass through the same workgroup.
#include "common.hpp"

namespace dlm {

typedef __attribute__((__vector_size__(4 * sizeof(short)))) short s16x4;
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
typedef __attribute__((__vector_size__(4 * sizeof(int)))) int i32x4;

struct BwdSeg {
    const uint16_t *k, *v;
    uint16_t *dk, *dv;
    int len, pos0;
    int64_t sb, sh, st;
    int rule;
};

struct BwdParams {
    int B, Lq, Hq, Hkv, g, R;
    const uint16_t *q, *o, *dout;
    int64_t q_sb, q_st, q_sh, o_sb, o_st, o_sh, do_sb, do_st, do_sh;
    uint16_t* dq;
    int64_t dq_sb, dq_st, dq_sh;
    BwdSeg seg[3];
    const float* lse;
    float* delta;
    int bs, q_pos0;
    float scale, scale_log2;
    const int32_t* cu;
    int total;
};

__device__ __forceinline__ bf16x8 bw_as_bf16x8(u32x4 v) {
    union { u32x4 u; bf16x8 b; } x;
    x.u = v;
    return x.b;
}

// index of (sequence b, head h, query row i) in the LSE / delta arrays; s0 = first token of the sequence (packed mode)
__device__ __forceinline__ int64_t stat_index(const BwdParams& p, int b, int h, int i, int s0) {
    return p.cu ? (int64_t)h * p.total + s0 + i : ((int64_t)b * p.Hq + h) * p.Lq + i;
}

// ---------------------------------------------------------------------------------------------------------
// -delta[b, h, i] = -sum_c dO * O, as the other kernels add it.  D / 8 lanes per row, 16-byte loads.
template <int D>
__global__ __launch_bounds__(256) void attn_bwd_delta_kernel(BwdParams p) {
    constexpr int LPR = D / 8;             // lanes per row
    constexpr int RPB = 256 / LPR;         // rows per workgroup
    const int b = blockIdx.z;
    int s0 = 0, sl = p.Lq;
    int64_t o_off = b * p.o_sb, do_off = b * p.do_sb;
    if (p.cu) {
        s0 = min(max(p.cu[b], 0), p.total);
        sl = max(min(min(p.cu[b + 1], p.total) - s0, p.Lq), 0);
        o_off = s0 * p.o_st;
        do_off = s0 * p.do_st;
    }
    const int row = blockIdx.x * RPB + threadIdx.x / LPR;   // row = i * Hq + h
    const int c = threadIdx.x % LPR;
    const int i = row / p.Hq, h = row - i * p.Hq;
    float acc = 0.f;
    if (i < sl) {
        const u32x4 a = *reinterpret_cast<const u32x4*>(p.o + o_off + i * p.o_st + (int64_t)h * p.o_sh + c * 8);
        const u32x4 d = *reinterpret_cast<const u32x4*>(p.dout + do_off + i * p.do_st + (int64_t)h * p.do_sh + c * 8);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            acc += bf16_bits_to_f32(a[e] & 0xffffu) * bf16_bits_to_f32(d[e] & 0xffffu);
            acc += bf16_bits_to_f32(a[e] >> 16) * bf16_bits_to_f32(d[e] >> 16);
        }
    }
#pragma unroll
    for (int off = LPR / 2; off >= 1; off >>= 1) acc += shfl_xor(acc, off);
    if (i < sl && c == 0) p.delta[stat_index(p, b, h, i, s0)] = -acc;
}

// ---------------------------------------------------------------------------------------------------------
template <int D, bool BC>
__global__ __launch_bounds__(256, 2) void attn_bwd_dq_kernel(BwdParams p, GridRemap rm) {
    constexpr int KP = D * 2 + 16;         // row-read image pitch (bytes)
    constexpr int TP = D * 2 + 64;         // transposing-read image pitch
    constexpr int C8 = D / 8;
    constexpr int NLD = (32 * C8) / 256;   // 16-byte chunks per thread per 32-row tile
    constexpr int OPB = D * 2 + 16;        // output staging row pitch (bytes)
    constexpr int TILES_BYTES = 2 * 32 * KP + 32 * TP, STAGE_BYTES = 4 * 32 * OPB + 4 * 32 * 8;
    __shared__ __attribute__((aligned(16))) unsigned char smem[TILES_BYTES > STAGE_BYTES ? TILES_BYTES : STAGE_BYTES];
    unsigned char* Krow = smem;
    unsigned char* Vrow = smem + 32 * KP;
    unsigned char* Ktr = smem + 2 * 32 * KP;

    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int n = lane & 31, hi = lane >> 5;
    int b = blockIdx.z, kvh = blockIdx.y, bx0 = blockIdx.x;
    if (rm.nx > 0) {
        int grp;
        if (!remap_decode(rm, p.B * p.Hkv, grp, bx0)) return;
        kvh = grp % p.Hkv;
        b = grp / p.Hkv;
    }
    const int r0 = bx0 * 128;

    int len0 = p.seg[0].len, len1 = p.seg[1].len, len2 = p.seg[2].len;
    int R = p.R, s0 = 0;
    int64_t q_off = b * p.q_sb, do_off = b * p.do_sb, dq_off = b * p.dq_sb, kv1_off = b * p.seg[1].sb;
    if (p.cu) {
        s0 = min(max(p.cu[b], 0), p.total);
        const int sl = max(min(min(p.cu[b + 1], p.total) - s0, p.Lq), 0);
        R = p.g * sl;
        if (r0 >= R) return;
        len1 = min(len1, sl);
        q_off = s0 * p.q_st;
        do_off = s0 * p.do_st;
        dq_off = s0 * p.dq_st;
        kv1_off = s0 * p.seg[1].st;
    }
    int F0 = 0, F1 = 0, F2 = 0, ho0 = 0, ho1 = 0, ho2 = 0;
    bool same0 = false, same1 = false, same2 = false;
    if (BC) {
        const int rows_end = min(r0 + 128, R);
        const int lim = ((p.q_pos0 + (rows_end - 1) / p.g) / p.bs + 1) * p.bs;
        const int first = ((p.q_pos0 + r0 / p.g) / p.bs) * p.bs;
        ho0 = (p.seg[0].rule == DLM_SEG_EARLIER_BLOCKS) ? p.bs : 0;
        ho1 = (p.seg[1].rule == DLM_SEG_EARLIER_BLOCKS) ? p.bs : 0;
        ho2 = (p.seg[2].rule == DLM_SEG_EARLIER_BLOCKS) ? p.bs : 0;
        same0 = p.seg[0].rule == DLM_SEG_SAME_BLOCK;
        same1 = p.seg[1].rule == DLM_SEG_SAME_BLOCK;
        same2 = p.seg[2].rule == DLM_SEG_SAME_BLOCK;
        len0 = max(0, min(len0, lim - ho0 - p.seg[0].pos0));
        len1 = max(0, min(len1, lim - ho1 - p.seg[1].pos0));
        len2 = max(0, min(len2, lim - ho2 - p.seg[2].pos0));
        if (same0) F0 = min(max(first - p.seg[0].pos0, 0) >> 5, (len0 + 31) >> 5);
        if (same1) F1 = min(max(first - p.seg[1].pos0, 0) >> 5, (len1 + 31) >> 5);
        if (same2) F2 = min(max(first - p.seg[2].pos0, 0) >> 5, (len2 + 31) >> 5);
    }
    const int T0 = ((len0 + 31) >> 5) - F0, T1 = ((len1 + 31) >> 5) - F1, T2 = ((len2 + 31) >> 5) - F2;
    const int T = T0 + T1 + T2;

    const uint16_t* kb0 = p.seg[0].k + b * p.seg[0].sb + kvh * p.seg[0].sh;
    const uint16_t* vb0 = p.seg[0].v + b * p.seg[0].sb + kvh * p.seg[0].sh;
    const uint16_t* kb1 = p.seg[1].k + kv1_off + kvh * p.seg[1].sh;
    const uint16_t* vb1 = p.seg[1].v + kv1_off + kvh * p.seg[1].sh;
    const uint16_t* kb2 = p.seg[2].k + b * p.seg[2].sb + kvh * p.seg[2].sh;
    const uint16_t* vb2 = p.seg[2].v + b * p.seg[2].sb + kvh * p.seg[2].sh;
    const int64_t st0 = p.seg[0].st, st1 = p.seg[1].st, st2 = p.seg[2].st;
    const int sp0 = __builtin_amdgcn_readfirstlane(p.seg[0].pos0), sp1 = __builtin_amdgcn_readfirstlane(p.seg[1].pos0),
              sp2 = __builtin_amdgcn_readfirstlane(p.seg[2].pos0);

    // ---- this lane's query row: Q and dO fragments (B operands), LSE and delta ----------------------------
    // All requested at once and unconditionally (a row past the end repeats the last one, gets no probability and is not stored): behind branches each
    // piece, and then LSE and delta, was a trip of its own.  Forward and backward, us: 4 x 777 tokens, block diffusion, 14/2 heads of 64 262 / 254.
    const bool valid = r0 + w * 32 + n < R;
    const int r = min(r0 + w * 32 + n, R - 1);
    const int qi = r / p.g;
    const int hg = r - qi * p.g;
    const int h = kvh * p.g + hg;
    bf16x8 qf[D / 16], dof[D / 16];
    const uint16_t* qp = p.q + q_off + qi * p.q_st + (int64_t)h * p.q_sh;
    const uint16_t* dp = p.dout + do_off + qi * p.do_st + (int64_t)h * p.do_sh;
#pragma unroll
    for (int c = 0; c < D / 16; ++c) {
        qf[c] = bw_as_bf16x8(*reinterpret_cast<const u32x4*>(qp + 16 * c + 8 * hi));
        dof[c] = bw_as_bf16x8(*reinterpret_cast<const u32x4*>(dp + 16 * c + 8 * hi));
    }
    const int64_t si = stat_index(p, b, h, qi, s0);
    const float row_lse = p.lse[si], delta = -p.delta[si];
    // +inf: every probability of an absent row (or one that saw no key) is 0
    const float lse2 = valid && row_lse > -INFINITY ? row_lse * 1.4426950408889634f : INFINITY;
    const int qlim = BC ? ((p.q_pos0 + qi) / p.bs + 1) * p.bs : 0;
    int qlim_min = 0x7fffffff, qlim_max = 0;
    if (BC) {
        qlim_min = qlim_max = qlim;
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
            qlim_min = min(qlim_min, shfl_xor(qlim_min, off));
            qlim_max = max(qlim_max, shfl_xor(qlim_max, off));
        }
        qlim_min = __builtin_amdgcn_readfirstlane(qlim_min);
        qlim_max = __builtin_amdgcn_readfirstlane(qlim_max);
    }

    f32x16 dq[D / 32];
#pragma unroll
    for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
        for (int i = 0; i < 16; ++i) dq[dt][i] = 0.f;

    u32x4 kreg[NLD], vreg[NLD];
#define BW_TILE(t, sg, lt, slen)                                                                         \
    const int sg = ((t) < T0) ? 0 : (((t) < T0 + T1) ? 1 : 2);                                           \
    const int lt = ((t) < T0) ? (t) + F0 : (((t) < T0 + T1) ? (t) - T0 + F1 : (t) - T0 - T1 + F2);      \
    const int slen = (sg == 0) ? len0 : ((sg == 1) ? len1 : len2);
#define BW_FETCH(t)                                                                                      \
    {                                                                                                    \
        const int tc_ = min((t), T - 1);                                                                 \
        BW_TILE(tc_, sg_, lt_, slen_)                                                                    \
        const uint16_t* kb = (sg_ == 0) ? kb0 : ((sg_ == 1) ? kb1 : kb2);                                \
        const uint16_t* vb = (sg_ == 0) ? vb0 : ((sg_ == 1) ? vb1 : vb2);                                \
        const int64_t stt = (sg_ == 0) ? st0 : ((sg_ == 1) ? st1 : st2);                                 \
        _Pragma("unroll") for (int q = 0; q < NLD; ++q) {                                                \
            const int cidx = tid + q * 256;                                                              \
            const int row = cidx / C8, c = cidx - row * C8;                                              \
            const int loc = min(lt_ * 32 + row, slen_ - 1);                                              \
            const int64_t off = loc * stt + c * 8;                                                       \
            kreg[q] = *reinterpret_cast<const u32x4*>(kb + off);                                         \
            vreg[q] = *reinterpret_cast<const u32x4*>(vb + off);                                         \
        }                                                                                                \
    }
#define BW_STORE(t)                                                                                      \
    {                                                                                                    \
        BW_TILE((t), sg_, lt_, slen_)                                                                    \
        (void)sg_;                                                                                       \
        _Pragma("unroll") for (int q = 0; q < NLD; ++q) {                                                \
            const int cidx = tid + q * 256;                                                              \
            const int row = cidx / C8, c = cidx - row * C8;                                              \
            const bool live = lt_ * 32 + row < slen_;                                                    \
            const u32x4 z = {0, 0, 0, 0};                                                                \
            const u32x4 kk = live ? kreg[q] : z;                                                         \
            *reinterpret_cast<u32x4*>(Krow + row * KP + c * 16) = kk;                                    \
            *reinterpret_cast<u32x4*>(Ktr + row * TP + c * 16) = kk;                                     \
            *reinterpret_cast<u32x4*>(Vrow + row * KP + c * 16) = live ? vreg[q] : z;                    \
        }                                                                                                \
    }

    if (T > 0) BW_FETCH(0);
    for (int t = 0; t < T; ++t) {
        BW_STORE(t);
        __syncthreads();
        BW_FETCH(t + 1);   // clamped to the last tile: the load is unconditional, its result unused past the end
        f32x16 S, dP;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            S[i] = 0.f;
            dP[i] = 0.f;
        }
#pragma unroll
        for (int c = 0; c < D / 16; ++c) {
            const bf16x8 kf = *reinterpret_cast<const bf16x8*>(Krow + n * KP + (16 * c + 8 * hi) * 2);
            const bf16x8 vf = *reinterpret_cast<const bf16x8*>(Vrow + n * KP + (16 * c + 8 * hi) * 2);
            S = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[c], S, 0, 0, 0);
            dP = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, dof[c], dP, 0, 0, 0);
        }
        BW_TILE(t, sg, lt, slen)
        const int spos0 = ((sg == 0) ? sp0 : ((sg == 1) ? sp1 : sp2)) + lt * 32;
        const int hoff = (sg == 0) ? ho0 : ((sg == 1) ? ho1 : ho2);
        const bool same = (sg == 0) ? same0 : ((sg == 1) ? same1 : same2);
        const bool ragged = (lt * 32 + 32 > slen) ||
                            (BC && (spos0 + 31 >= qlim_min - hoff || (same && spos0 < qlim_max - p.bs)));
        if (ragged) {
            const int pbase = spos0 + 4 * hi;
            int hi_r = spos0 - lt * 32 + slen;
            int lo_r = -(1 << 30);
            if (BC) {
                hi_r = min(hi_r, qlim - hoff);
                if (same) lo_r = qlim - p.bs;
            }
            const unsigned span = (unsigned)max(hi_r - lo_r, 0);
            const unsigned off0 = (unsigned)(pbase - lo_r);
#pragma unroll
            for (int i = 0; i < 16; ++i)
                if (off0 + (unsigned)(8 * (i >> 2) + (i & 3)) >= span) S[i] = -INFINITY;
        }
        uint32_t pk[8];
#pragma unroll
        for (int i = 0; i < 16; i += 2) {
            const float p0 = fast_exp2(fmaf(S[i], p.scale_log2, -lse2));
            const float p1 = fast_exp2(fmaf(S[i + 1], p.scale_log2, -lse2));
            pk[i >> 1] = pack_bf16x2(p0 * (dP[i] - delta), p1 * (dP[i + 1] - delta));
        }
        bf16x8 dsf[2];
        {
            u32x4 lo = {pk[0], pk[1], pk[2], pk[3]}, hi4 = {pk[4], pk[5], pk[6], pk[7]};
            dsf[0] = bw_as_bf16x8(lo);
            dsf[1] = bw_as_bf16x8(hi4);
        }
        const int s16 = lane & 15, blk = (lane >> 4) & 1;
#pragma unroll
        for (int dt = 0; dt < D / 32; ++dt) {
#pragma unroll
            for (int j2 = 0; j2 < 2; ++j2) {
                union { s16x4 h[2]; bf16x8 v; } kt;
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const int krow = 16 * j2 + 8 * q + 4 * hi + (s16 >> 2);
                    const int dcol = 32 * dt + 16 * blk + 4 * (s16 & 3);
                    kt.h[q] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(Ktr + krow * TP + dcol * 2));
                }
                dq[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kt.v, dsf[j2], dq[dt], 0, 0, 0);
            }
        }
        __syncthreads();
    }
#undef BW_TILE
#undef BW_FETCH
#undef BW_STORE

    // dQ^T sits in the accumulators with lane = row: each wavefront transposes its 32 rows through a private LDS
    // region (the tiles are dead: the loop ended with a barrier, or never ran) and stores whole rows, 16 bytes per
    // lane, instead of 64 stores that touch 32 rows with 16 bytes each.
    {
        unsigned char* ob = smem + w * (32 * OPB);
        int64_t* roff = reinterpret_cast<int64_t*>(smem + 4 * 32 * OPB) + w * 32;
        if (hi == 0) roff[n] = valid ? qi * p.dq_st + (int64_t)h * p.dq_sh : (int64_t)-1;
#pragma unroll
        for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {
                u32x2 v;
                v[0] = pack_bf16x2(dq[dt][4 * q4] * p.scale, dq[dt][4 * q4 + 1] * p.scale);
                v[1] = pack_bf16x2(dq[dt][4 * q4 + 2] * p.scale, dq[dt][4 * q4 + 3] * p.scale);
                *reinterpret_cast<u32x2*>(ob + n * OPB + (32 * dt + 8 * q4 + 4 * hi) * 2) = v;
            }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // one wavefront's LDS operations complete in order
#pragma unroll
        for (int q = 0; q < (32 * C8) / 64; ++q) {
            const int id = q * 64 + lane;
            const int row = id / C8, c = id - row * C8;
            const int64_t ro = roff[row];
            const u32x4 v = *reinterpret_cast<const u32x4*>(ob + row * OPB + c * 16);
            if (ro >= 0) *reinterpret_cast<u32x4*>(p.dq + dq_off + ro + 8 * c) = v;
        }
    }
}

// ---------------------------------------------------------------------------------------------------------
// A 32-row tile image as the transposing and the row reads both want it: requests of 1024 bytes (4 rows at d = 128, 8 at
// d = 64) sit 1040 bytes apart, and inside a request piece c (16 bytes) of row r is stored in place c ^ bw_swz(r).  Row
// reads (16 rows, one piece each) and transposing reads (4 rows x 64 bytes) then touch every bank once, and
// global_load_lds, whose lanes fill 16-byte places in order, can write it.  The exclusive-or moves only 64-byte (d = 128)
// or 32-byte (d = 64) steps, so 4 lane addresses serve all row reads of a tile and 4 or 2 all transposing ones.
constexpr int BW_GP = 1040;
template <int D>
__device__ __forceinline__ int bw_swz(int row) {
    return D == 128 ? (row & 3) << 2 : (((row >> 1) & 1) << 2) | (((row >> 2) & 1) << 1);
}

// i * stride, without the 64-bit product: a stride outside 32 bits leaves room for fewer than 2^23 rows in any memory, so
// its upper part takes a 24-bit product
__device__ __forceinline__ int64_t bw_offset(int i, int64_t stride) {
    const int32_t lo = (int32_t)stride;
    const int hi = (int)((stride - lo) >> 32);
    return (int64_t)i * lo + ((int64_t)__mul24(i, hi) << 32);
}

// Memory to LDS, 16 or 4 bytes a lane, to consecutive places from a wave-uniform address on.  Asm, so that the compiler, which
// cannot tell the ring's stages apart, does not wait for every request in flight before each transposing read; the
// waits that are needed stand in the loop.  No registers are written.
// Where the compiler takes a scalar operand from (it may be restored from a spill by a lane read right in front of the block) is not
// known here, and a vector instruction has to stay two wait states behind a lane read of its scalar, a memory address
// five.  So scalar operands are read by scalar instructions alone, for which the hardware waits, and addresses are what those wrote.
__device__ __forceinline__ void bw_load_lds16(const void* src, uint32_t dst) {
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(src), "s"(__builtin_amdgcn_readfirstlane(dst)) : "memory");
}
// the same 16 bytes a lane at offset + delta of two operands (base0, base1: wave-uniform), to dst and dst + GAP
template <int GAP>
__device__ __forceinline__ void bw_load_lds16_pair(const void* base0, const void* base1, uint32_t offset, uint32_t delta, uint32_t dst) {
    uint64_t a;
    asm volatile("s_mov_b32 m0, %2\n\ts_mov_b64 %0, %3\n\tglobal_load_lds_dwordx4 %1, %0\n\ts_add_u32 m0, %2, %5\n\ts_mov_b64 %0, %4\n\tglobal_load_lds_dwordx4 %1, %0"
                 : "=&s"(a) : "v"(offset), "s"(__builtin_amdgcn_readfirstlane(dst)), "s"((uintptr_t)base0 + delta), "s"((uintptr_t)base1 + delta), "n"(GAP) : "memory", "scc");
}
__device__ __forceinline__ void bw_load_lds16(const void* base, uint32_t offset, uint32_t dst) {   // base: wave-uniform
    uint64_t a;
    asm volatile("s_mov_b32 m0, %2\n\ts_mov_b64 %0, %3\n\tglobal_load_lds_dwordx4 %1, %0"
                 : "=&s"(a) : "v"(offset), "s"(__builtin_amdgcn_readfirstlane(dst)), "s"(base) : "memory");
}
__device__ __forceinline__ void bw_load_lds4(const void* src, uint32_t dst) {
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dword %0, off" ::"v"(src), "s"(__builtin_amdgcn_readfirstlane(dst)) : "memory");
}

// c += a * b with c in accumulation registers.  Written as asm because the compiler gives all matrix results of a
// function one register class: in accumulation registers the scores would be copied back before every exponential.
// fresh (a constant): b may just have been written by a vector instruction, which the product has to stay two wait states behind.
__device__ __forceinline__ void bw_mfma_acc(f32x16& c, bf16x8 a, bf16x8 b, bool fresh) {
    if (fresh) asm volatile("s_nop 1\n\tv_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(a), "v"(b));
    else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(a), "v"(b));
}

// c = a * b (the first product of a chain: no register is zeroed for it).  The next reader of c is another product with one
// in between, or far behind; s_nop as above, should the compiler have to move an operand into place.
__device__ __forceinline__ void bw_mfma_zero(f32x16& c, bf16x8 a, bf16x8 b) {
    asm volatile("s_nop 1\n\tv_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(c) : "v"(a), "v"(b));
}

// Is a workgroup ever given two slabs (`pair`)?  Only with two wavefronts side by side: one has one slab in all, and where wavefronts share a slab's rows
// there are hardly slabs enough for it.  Without the second pass nothing has to be kept over the first (8 x 2048 tokens, blocks of 32, 4 heads of 64, forward
// and backward: 521 -> 494 us).
template <bool BC, int NWK, int NWR>
constexpr bool dkv_pairs() { return BC && NWK == 2 && NWR == 1; }

// the lane number, formed where it stands (asm: what follows from it is not moved away or kept in registers in its place)
__device__ __forceinline__ int bw_lane() {
    int l = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0));
    asm volatile("" : "+v"(l));
    return l;
}

// Strides of Q and dO of less than 2^24 bytes, all of a group's heads within 2^30: requests can take 32-bit offsets
__host__ __device__ __forceinline__ bool small_strides(const BwdParams& p) {
    return p.q_st >= 0 && p.q_sh >= 0 && p.do_st >= 0 && p.do_sh >= 0 && p.q_st < (1 << 23) && p.q_sh < (1 << 23) &&
           p.do_st < (1 << 23) && p.do_sh < (1 << 23) && p.g * p.q_sh < (1 << 29) && p.g * p.do_sh < (1 << 29);
}

// dK and dV of one segment in one pass.  A wavefront owns 64 keys (two MFMA column tiles, K and V fragments and both
// accumulators in registers) and walks 32-row tiles of (query, head in group) rows; NWK wavefronts side by side share
// the tiles through LDS, NWR groups of them take every NWR-th tile and are summed through LDS at the end.
//
// What bounds it: every MFMA's A operand (Q, dO rows, dO^T, Q^T) comes from LDS, 32 KB per wavefront and tile.  With 32
// keys a wavefront that is one 1 KB fragment per MFMA, all that the LDS delivers at full MFMA rate; 64 keys use each
// fragment twice.  That takes the whole register file (one wavefront per SIMD), so nothing may wait in turn:
//   * S is formed once for dV and dK (two passes, one for each, formed it twice: 5 products instead of 4);
//   * the exponentials sit between the MFMAs of dP and of the first half of dV, dS between those of the second half of
//     dV and the first of dK (there is one wavefront a SIMD: only its own vector and matrix instructions can overlap);
//   * tiles go from memory to LDS without registers (global_load_lds) through a ring of four, two tiles ahead, and the
//     next tile's first fragments are read before this tile's last MFMAs: the barrier sits between;
//   * one wavefront issues one instruction at a time: 3.9 vector and 2.3 scalar instructions per MFMA, after 7.5 and 1.7 with
//     LDS addresses, row divisions and statistics formed per read (2.6 -> 1.9 ms below).  The compiler still spills 30 - 70 scalars
//     to lanes of vector registers, the more the more request paths a kernel has (ALIKE), some of which come back every tile;
//   * nothing covers what a workgroup does before its first product, so K, V and the first tiles travel together: no vector register is
//     spilled in the shapes that large launches take (with 18 or 50 of them kept on the stack from the start of the kernel on, every reload
//     waited for all requests before it: five trips to memory one after another, 1.72 -> 1.63 ms on the packed batch below).
// Measured (8 x 4096 tokens, 32 / 8 heads of 128, blocks of 4): 1.86 - 1.95 ms = 1.17 PFLOP/s of products, two passes with 32
// keys a wavefront 4.28 ms; 128 packed sequences of 64 k tokens, 32 heads: 1.63 ms, two passes 2.86.  MFMA pipes busy 0.52 at
// 2.2 GHz: with all loads, waits and vector work taken out the loop still runs at 1.35 PFLOP/s, the power limit on such data.
template <int D, bool BC, int NWK, int NWR, bool ALIKE>
__global__ __launch_bounds__(64 * NWK * NWR, 1) void attn_bwd_dkv_kernel(BwdParams p, int sidx, int n_slabs, int pair, GridRemap rm) {
    constexpr bool PAIR = dkv_pairs<BC, NWK, NWR>();   // a workgroup may take two slabs
    constexpr int NS = D == 128 && NWK * NWR == 1 ? 2 : 4;   // ring stages: four such rings fit a CU, one a SIMD
    constexpr int FD = D == 128 ? 2 : 4;               // fragments read ahead (at d = 128 all that registers allow)
    constexpr int AHEAD = NWK == 1 ? NS - 1 : 2;       // tiles requested ahead: a ring that is the wavefront's own needs no slack
    constexpr int P = D * 2, C8 = D / 8;
    constexpr int RPI = 64 / C8, IPW = 32 / RPI / NWK; // rows per request, requests per wavefront, operand and tile
    constexpr int IMG = 32 / RPI * BW_GP;              // one operand's tile image
    constexpr int STAGE = 2 * IMG;                     // Q, dO
    constexpr int LOADS = 2 * IPW + 1;                 // ... with the statistics
    constexpr int KS = 64 * NWK;                       // keys per workgroup
    constexpr int OPB = D * 2 + 16;                    // output staging row pitch (bytes)
    constexpr int RING = NWR * NS * STAGE;
    constexpr int MERGE = NWR > 1 ? NWK * 64 * D * 4 : 0;
    constexpr int STORE = NWK * 32 * OPB;
    constexpr int BODY = RING > MERGE ? (RING > STORE ? RING : STORE) : (MERGE > STORE ? MERGE : STORE);
    static_assert(BODY + NWK * NWR * NS * 256 <= 160 * 1024, "LDS");
    static_assert(IPW >= 1, "at least one request per wavefront");
    __shared__ __attribute__((aligned(1024))) unsigned char smem[BODY + NWK * NWR * NS * 256];

    const int tid = threadIdx.x;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wk = w % NWK, wr = w / NWK;
    int b = blockIdx.z, kvh = blockIdx.y, bx = blockIdx.x;
    if (rm.nx > 0) {
        int grp;
        if (!remap_decode(rm, p.B * p.Hkv, grp, bx)) return;
        kvh = grp % p.Hkv;
        b = grp / p.Hkv;
    }
    // plain locals per segment field (a dynamically indexed struct member would go through memory)
    const uint16_t* sk = (sidx == 0) ? p.seg[0].k : ((sidx == 1) ? p.seg[1].k : p.seg[2].k);
    const uint16_t* sv = (sidx == 0) ? p.seg[0].v : ((sidx == 1) ? p.seg[1].v : p.seg[2].v);
    uint16_t* sdk = (sidx == 0) ? p.seg[0].dk : ((sidx == 1) ? p.seg[1].dk : p.seg[2].dk);
    uint16_t* sdv = (sidx == 0) ? p.seg[0].dv : ((sidx == 1) ? p.seg[1].dv : p.seg[2].dv);
    int slen = (sidx == 0) ? p.seg[0].len : ((sidx == 1) ? p.seg[1].len : p.seg[2].len);
    const int spos = (sidx == 0) ? p.seg[0].pos0 : ((sidx == 1) ? p.seg[1].pos0 : p.seg[2].pos0);
    const int64_t ssb = (sidx == 0) ? p.seg[0].sb : ((sidx == 1) ? p.seg[1].sb : p.seg[2].sb);
    const int64_t ssh = (sidx == 0) ? p.seg[0].sh : ((sidx == 1) ? p.seg[1].sh : p.seg[2].sh);
    const int64_t sst = (sidx == 0) ? p.seg[0].st : ((sidx == 1) ? p.seg[1].st : p.seg[2].st);
    const int srule = (sidx == 0) ? p.seg[0].rule : ((sidx == 1) ? p.seg[1].rule : p.seg[2].rule);

    int s0 = 0, Lq = p.Lq;
    int64_t q_off = b * p.q_sb, do_off = b * p.do_sb, kv_off = b * ssb;
    if (p.cu) {
        s0 = min(max(p.cu[b], 0), p.total);
        const int sl = max(min(min(p.cu[b + 1], p.total) - s0, p.Lq), 0);
        Lq = sl;
        slen = min(slen, sl);
        q_off = s0 * p.q_st;
        do_off = s0 * p.do_st;
        kv_off = s0 * sst;
    }
    const int hoff = (BC && srule == DLM_SEG_EARLIER_BLOCKS) ? p.bs : 0;
    const bool same = BC && srule == DLM_SEG_SAME_BLOCK;
    // requests with 32-bit offsets from a wave-uniform query
    const bool small = ALIKE || small_strides(p);
    const bool alike = ALIKE || (small && p.q_st == p.do_st && p.q_sh == p.do_sh);
    const int64_t do_st = ALIKE ? p.q_st : p.do_st, do_sh = ALIKE ? p.q_sh : p.do_sh;
    // Rows in order of (query, head), or (by_head) the queries of one head after another, each head cut into tiles of its own: where the heads do not
    // divide a tile, the place of a row in it changes from tile to tile, and forming it costs some 30 vector instructions a request (see
    // `regular`).  With the heads apart a tile is 32 queries of one head whatever their number.  Where that makes at most an eighth more
    // tiles (a head's last tile is partly empty).  Forward and backward, us, before / with it and ALIKE: 64 packed sequences of 48 - 900 tokens, 14/2
    // heads of 64 504 / 471, 4 x 777 tokens, block diffusion 301 / 262; 28/4 heads of 128, 1425 / 1325.
    const bool by_head = ALIKE && (32 % p.g) != 0 && 8 * p.g * ((Lq + 31) >> 5) <= 9 * ((p.g * Lq + 31) >> 5);
    const int g = by_head ? 1 : p.g;                   // heads that the rows of a tile run over
    const int R = g * Lq;
    // Row r of the group is query r / g, head r % g.  Inside a tile that starts at (query i0, head h0) row l is on query i0 + 1 + u / g
    // rounded down, u = h0 + l - g: on i0 where u < 0, and otherwise u < 31, where u * ceil(2^16 / g) / 2^16 rounds down to the same (the
    // excess is below 31 / 2^16, u / g at least 1 / 31 short of the next whole number, or g > 31 and both are 0).
    const int mul_g = (65536 + g - 1) / g;
    const uint16_t* const qb = p.q + q_off + (int64_t)(kvh * p.g) * p.q_sh;
    const uint16_t* const gb = p.dout + do_off + (int64_t)(kvh * p.g) * p.do_sh;
    const int st_h = p.cu ? p.total : p.Lq;            // statistics of the next head
    const int stat_base = BODY + w * NS * 256;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;

    // The usual case: 1, 2, 4 .. 32 heads a tile and Q and dO laid out alike.  A tile then holds whole queries, so row l of any
    // tile is at the same place relative to its first row: one lane offset, and a wave-uniform step from request to request.
    // (Per row this is 1 vector instruction for both operands instead of some 20.)
    const bool regular = alike && (32 % g) == 0;
    const int gsh = 31 - __builtin_clz(g);
    const int qst2 = (int)p.q_st * 2, qsh2 = (int)p.q_sh * 2;

    // Under a block-causal mask the work of a key slab shrinks with its index (later keys are seen by fewer rows).
    // pair != 0: a workgroup takes slab x and then slab n_slabs - 1 - x, so every workgroup does the same amount
    // of work and the workgroups of one (sequence, KV head) stay in step on the same Q / dO tiles (L2 reuse).
    // pair == 0: one slab per workgroup; every second group of 8 slabs is taken in reverse so that the 8 XCDs,
    // which get workgroups round-robin, receive equal sums.
#pragma clang loop unroll(disable)
    for (int pass = 0; pass < (PAIR && pair ? 2 : 1); ++pass) {
    int slab = bx;
    if (PAIR && pair) {
        slab = pass ? n_slabs - 1 - bx : bx;
        if (pass && slab <= bx) break;
    } else {
        const int oct = bx >> 3;
        if ((oct & 1) && (oct * 8 + 7 < n_slabs)) slab = oct * 8 + 7 - (bx & 7);
    }
    const int j0 = slab * KS;                         // first key of this pass inside the segment
    if (j0 >= slen) continue;
    const int jw = j0 + wk * 64;                      // first key of this wavefront (past the end: nothing to multiply)

    // What depends on the lane is formed anew here, not kept in registers from one pass to the next (they were spilled, and every reload
    // waited for the requests in flight)
    const int lane = bw_lane();
    const int n = lane & 31, hi = lane >> 5;

    // ---- this lane's two keys: K and V fragments (B operands).  A key past the end repeats the last one; its column
    // of the accumulators is never stored. --------------------------------------------------------------------------
    bf16x8 kf[2][D / 16], vf[2][D / 16];
    int r_clear_lo = 0, r_clear_hi = R;               // rows that see every key of the wavefront
    int r_first = 0;                                  // no row before it sees any
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const int j = jw + 32 * s + n;
        const int64_t ko = kv_off + kvh * ssh + (int64_t)min(j, slen - 1) * sst;
#pragma unroll
        for (int c = 0; c < D / 16; ++c) {
            kf[s][c] = bw_as_bf16x8(*reinterpret_cast<const u32x4*>(sk + ko + 16 * c + 8 * hi));
            vf[s][c] = bw_as_bf16x8(*reinterpret_cast<const u32x4*>(sv + ko + 16 * c + 8 * hi));
        }
    }
    // lane parts of the LDS addresses: row reads (row n, piece 2 c + hi) and transposing reads (row 16 j + 8 q + 4 hi + s16 / 4,
    // piece 4 dt + 2 blk + ...); the step-dependent part is an exclusive-or above bit 5 or 6
    constexpr int RSH = D == 128 ? 6 : 5, RDIV = D == 128 ? 2 : 1;
    const int row_base = n / RPI * BW_GP + n % RPI * P + hi * 16;
    const int row_x = bw_swz<D>(n) >> 1 << 5 & (D == 128 ? 0xc0 : 0x60);
    const int s16 = lane & 15, blk = (lane >> 4) & 1;
    const int tr_base = (D == 128 ? hi * BW_GP + (s16 >> 2) * P : (4 * hi + (s16 >> 2)) * P) +
                        (((2 * blk + ((s16 & 3) >> 1)) ^ (D == 128 ? 0 : 2 * hi)) << 4) + 8 * (s16 & 1);
    const int tr_x = (D == 128 ? s16 >> 2 : s16 >> 3) << 6;
    // statistics: lanes 0..31 fetch LSE, lanes 32..63 delta of the tile's rows
    const float* const stp = (hi ? p.delta : p.lse) + stat_index(p, b, kvh * p.g, 0, s0);
    const uint32_t voff = regular ? __umul24((lane / C8) >> gsh, qst2) + __umul24((lane / C8) & (g - 1), qsh2) + ((lane % C8) ^ bw_swz<D>(lane / C8)) * 16 : 0;
    const float* const sptr = stp + (int64_t)(n & (g - 1)) * st_h + (n >> gsh);
    // ---- rows that can see some key of this workgroup: tiles [rt_begin, rt_end) -----------------------------
    int rt_begin = 0, rt_end = (R + 31) >> 5;
    if (BC) {
        const int kp_first = spos + j0, kp_last = spos + min(j0 + KS - 1, slen - 1);
        const int i_begin = max(0, ((kp_first + hoff) / p.bs) * p.bs - p.q_pos0);
        rt_begin = min(rt_end, (int)(((int64_t)i_begin * g) >> 5));
        if (same) {
            const int i_end = max(0, min(Lq, (kp_last / p.bs + 1) * p.bs - p.q_pos0));
            rt_end = max(rt_begin, min(rt_end, (i_end * g + 31) >> 5));
        }
        const int kw_first = spos + jw, kw_last = spos + jw + 63;
        r_clear_lo = min(max((kw_last + hoff) / p.bs * p.bs - p.q_pos0, 0), Lq) * g;
        if (same) r_clear_hi = min(max((kw_first + p.bs) / p.bs * p.bs - p.q_pos0, 0), Lq) * g;
        r_first = min(max((kw_first + hoff) / p.bs * p.bs - p.q_pos0, 0), Lq) * g;
    }
    const int n_rt = rt_end - rt_begin;
    const int n_tiles = by_head ? n_rt * p.g : n_rt;
    const int n_it = (n_tiles + NWR - 1) / NWR;

    // Row tiles are walked from the last one down: under a block-causal mask the workgroups of one (sequence,
    // KV head) differ in where their range BEGINS, so this way they all start on the same tile and stay in step.
    // The second slab of a pair is walked upwards: its range begins where the first slab's walk ended (slab x ends
    // after n - x steps, slab n - 1 - x begins at tile n - 1 - x), so at any time all the workgroups of the group
    // that are in their second pass are on one tile again, whatever their x.
    const bool up = PAIR && pair && pass;
    int rt = up ? rt_begin + wr : rt_end - 1 - wr;    // this wavefront's tile (by_head: of one head, over and over)
#define BW_WRAP() if (ALIKE && by_head && n_rt > 0) { while (rt < rt_begin) rt += n_rt; while (rt >= rt_end) rt -= n_rt; }
    const int rt_step = up ? NWR : -NWR;

    // next tile to request: first row = query i0, head h0 (kept without divisions); queries are clamped to the sequence,
    // so a request past either end of the walk reads rows that exist and that nobody multiplies
    int i0, h0;
    {
        const int r = rt * 32;
        i0 = __builtin_amdgcn_readfirstlane(r >= 0 ? r / g : -((-r + g - 1) / g));
        h0 = __builtin_amdgcn_readfirstlane(r - i0 * g);
    }
    const int di = 32 * NWR / g, dh = 32 * NWR - di * g;
    int ist = 0;                                      // ring stage it goes to
    // regular tiles: its first row of Q and of dO, and the step to the next tile's; whole: all 32 rows exist
    const int qpt = regular ? 32 >> gsh : 0;
    const uint16_t *qt = qb + (regular ? i0 * p.q_st : 0), *gt = gb + (regular ? i0 * p.q_st : 0);
    const int64_t dqt = regular ? (up ? di : -di) * p.q_st : 0;
    // by_head: head that the request cursor is on (requests past the end stay on the last one), its part of the statistics' address; after a head's last
    // tile the cursor goes back to the first tile's place, a head further
    int hd = 0;
    int64_t hstat = 0;
#define BW_NEXT_HEAD()                                                                                   \
    if (ALIKE && by_head && n_rt > 0) {                                                                \
        while (i0 < rt_begin * 32 || i0 >= rt_end * 32) {                                                \
            const int back_ = i0 < rt_begin * 32 ? n_rt * 32 : -n_rt * 32;                               \
            const int64_t dh_ = hd + 1 < p.g ? p.q_sh : 0;                                               \
            i0 += back_;                                                                                 \
            qt += back_ * p.q_st + dh_;                                                                  \
            gt += back_ * p.q_st + dh_;                                                                  \
            if (hd + 1 < p.g) { ++hd; hstat += st_h; }                                                   \
        }                                                                                                \
    }
    BW_NEXT_HEAD()
    BW_WRAP()
    bool whole = regular && i0 >= 0 && i0 + qpt <= Lq;
#define BW_ROW(l, i_, h_)                                                                                \
    const int u_ = h0 - g + (l);                                                                         \
    const int dv_ = __mul24(max(u_, -1), mul_g) >> 16;                                                   \
    const int h_ = u_ - dv_ * g;                                                                         \
    const int i_ = min(max(i0 + 1 + dv_, 0), Lq - 1);
    // request x of a tile: x < IPW a group of Q rows and the same dO rows, x == IPW the statistics.  The lane number is made
    // opaque, so that the offsets are formed anew for each tile instead of being kept in registers the loop does not have.
#define BW_REQUEST(x)                                                                                    \
    {                                                                                                    \
        if ((x) < IPW) {                                                                                 \
            const int q_ = wk * IPW + (x);                                                               \
            const uint32_t dst_ = lds0 + (wr * NS + ist) * STAGE + q_ * BW_GP;                           \
            if (whole) {                                                                                 \
                bw_load_lds16_pair<IMG>(qt, gt, voff, ((q_ * RPI) >> gsh) * qst2 + ((q_ * RPI) & (g - 1)) * qsh2, dst_); \
            } else {                                                                                     \
            const unsigned lo_ = bw_lane();                                                              \
            const int c16 = ((int)(lo_ % C8) ^ bw_swz<D>(lo_ / C8)) * 16;                                \
            BW_ROW(q_ * RPI + (int)(lo_ / C8), i_, h_)                                                   \
            if (small) {                                                                                 \
                const int ic_ = min(max(i0, 0), Lq - 1);                                                 \
                const uint32_t oq_ = __umul24(i_ - ic_, (int)p.q_st * 2) + __umul24(h_, (int)p.q_sh * 2) + c16;   \
                const uint32_t og_ = ALIKE ? oq_ : __umul24(i_ - ic_, (int)do_st * 2) + __umul24(h_, (int)do_sh * 2) + c16; \
                bw_load_lds16(qb + ic_ * p.q_st + hd * p.q_sh, oq_, dst_);                               \
                bw_load_lds16(gb + ic_ * do_st + hd * do_sh, og_, dst_ + IMG);                           \
            } else {                                                                                     \
                bw_load_lds16(qb + bw_offset(i_, p.q_st) + bw_offset(h_, p.q_sh) + c16 / 2, dst_);       \
                bw_load_lds16(gb + bw_offset(i_, do_st) + bw_offset(h_, do_sh) + c16 / 2, dst_ + IMG); \
            }                                                                                            \
            }                                                                                            \
        } else if (whole) {                                                                              \
            bw_load_lds4(sptr + i0 + hstat, lds0 + stat_base + ist * 256);                               \
        } else {                                                                                         \
            const unsigned lo_ = bw_lane();                                                              \
            BW_ROW((int)(lo_ & 31), i_, h_)                                                              \
            bw_load_lds4(stp + hstat + (int64_t)h_ * st_h + i_, lds0 + stat_base + ist * 256);           \
        }                                                                                                \
    }
#define BW_ADVANCE()                                                                                     \
    {                                                                                                    \
        ist = ist + 1 == NS ? 0 : ist + 1;                                                               \
        if (up) { i0 += di; h0 += dh; if (h0 >= g) { h0 -= g; ++i0; } }                                  \
        else { i0 -= di; h0 -= dh; if (h0 < 0) { h0 += g; --i0; } }                                      \
        qt += dqt;                                                                                       \
        gt += dqt;                                                                                       \
        BW_NEXT_HEAD()                                                                                   \
        whole = regular && i0 >= 0 && i0 + qpt <= Lq;                                                    \
    }
    // fragment of step s (0 .. 4 * PH - 1): Q rows, dO rows, dO^T, Q^T; the transposed ones in the order keys 0..15, 16..31
    constexpr int PH = D / 16;                        // steps per product
    union Frag { s16x4 h[2]; bf16x8 v; };
#define BW_ROW_ADDR(a, sb) _Pragma("unroll") for (int k = 0; k < 4; ++k) a[k] = (row_x ^ (k << RSH)) + ((sb) + row_base);
#define BW_TR_ADDR(a, sb) _Pragma("unroll") for (int k = 0; k < D / 32; ++k) a[k] = (tr_x ^ (k << 6)) + ((sb) + tr_base);
#define BW_READ(f, ra, ta, s)                                                                            \
    {                                                                                                    \
        if ((s) < 2 * PH) {                                                                              \
            const int c_ = (s) % PH;                                                                     \
            f.v = *reinterpret_cast<const bf16x8*>(smem + ra[c_ / RDIV] + (c_ % RDIV) * 32 + ((s) < PH ? 0 : IMG)); \
        } else {                                                                                         \
            const int j2_ = ((s) % PH) / (D / 32), dt_ = (s) % (D / 32);                                 \
            _Pragma("unroll") for (int q = 0; q < 2; ++q)                                                \
                f.h[q] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(smem + ta[dt_] +           \
                             (2 * j2_ + q) * (8 / RPI) * BW_GP + ((s) < 3 * PH ? IMG : 0)));             \
        }                                                                                                \
    }

    Frag fr[FD];
    int st = 0;                                       // ring stage of this iteration's tile
    if (n_it > 0) {
#pragma unroll
        for (int a = 0; a < AHEAD; ++a) {
#pragma unroll
            for (int x = 0; x <= IPW; ++x) BW_REQUEST(x);
            BW_ADVANCE();
        }
    }
    f32x16 av[2][D / 32], ak[2][D / 32];   // dV^T, dK^T: lane = key, registers = 16 of the 32 head-dim entries of tile dt
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
            for (int i = 0; i < 16; ++i) av[s][dt][i] = ak[s][dt][i] = 0.f;
    // K, V and the first tiles: a full wait, after which the compiler counts no load of its own inside the loop
    __builtin_amdgcn_s_waitcnt(0x0F70);               // vmcnt(0)
    if (n_it > 0) {
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
#pragma unroll
        for (int s = 0; s < FD; ++s) {
            int ra[4], ta[D / 32];
            BW_ROW_ADDR(ra, wr * NS * STAGE)
            BW_READ(fr[s], ra, ta, s);
        }
    }
    for (int it = 0; it < n_it; ++it) {
        const int sb = (wr * NS + st) * STAGE;
        const int stn = st + 1 == NS ? 0 : st + 1;
        const int sbn = (wr * NS + stn) * STAGE;
        const bool work = jw < slen && it * NWR + wr < n_tiles && rt * 32 + 32 > r_first;
        int ra[4], ta[D / 32];                        // LDS addresses of the row and the transposing reads
        if (work) {
            BW_ROW_ADDR(ra, sb)
            float* const stat = reinterpret_cast<float*>(smem + stat_base + st * 256);
            f32x16 S[2], dP[2];
            uint32_t pk[2][8];                        // P, then dS, as bf16 pairs: the B operands of the last two products
            f32x4 l2, sr;                             // statistics in use and the next four
            const float own_lse = stat[n];            // of row n: for the check below
#pragma unroll
            for (int c = 0; c < PH; ++c) {
#pragma unroll
                for (int s = 0; s < 2; ++s) {         // S[row, key]: lane = key
                    if (c == 0) bw_mfma_zero(S[s], fr[0].v, kf[s][0]);
                    else S[s] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[c % FD].v, kf[s][c], S[s], 0, 0, 0);
                }
                BW_READ(fr[c % FD], ra, ta, c + FD);
                // the tile after the next goes into the stage that the tile before the last one has left
#pragma unroll
                for (int x = 0; x <= IPW; ++x)
                    if (x * PH / (IPW + 1) == c) BW_REQUEST(x);
                __builtin_amdgcn_sched_barrier(0);
            }
            // Hidden scores become -inf (probability 0), on the tiles that hold some: rows outside [r_clear_lo, r_clear_hi) miss
            // a key of this wavefront, rows from R on do not exist
            if (__any(!(own_lse > -INFINITY))) {      // rows that saw no key (or have no LSE: NaN) take +inf: probabilities 0
                if (hi == 0 && !(own_lse > -INFINITY)) stat[n] = INFINITY;
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // one wavefront's LDS operations complete in order
            }
            if (rt * 32 < r_clear_lo || rt * 32 + 32 > r_clear_hi) {
                const int lo = bw_lane();             // formed here, on these few tiles, not kept in registers over the loop
                const int rbase = rt * 32 + 4 * (lo >> 5);
#pragma unroll
                for (int s = 0; s < 2; ++s) {
                    int rlo = 0, rhi = R;             // rows that see the lane's key
                    if (BC) {
                        const int kpos = spos + jw + 32 * s + (lo & 31);
                        rlo = min(max((kpos + hoff) / p.bs * p.bs - p.q_pos0, 0), Lq) * g;
                        if (same) rhi = min(max((kpos + p.bs) / p.bs * p.bs - p.q_pos0, 0), Lq) * g;
                    }
                    const unsigned span = (unsigned)max(rhi - rlo, 0);
#pragma unroll
                    for (int i = 0; i < 16; ++i)
                        if ((unsigned)(rbase + 8 * (i >> 2) + (i & 3) - rlo) >= span) S[s][i] = -INFINITY;
                }
            }
            constexpr int MP = 2 * PH;                // MFMAs per product
            sr = *reinterpret_cast<const f32x4*>(stat + 4 * hi);
            // dP starts from -delta (what the workspace holds): dS = P * (dP - delta) is one multiplication
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
                for (int g4 = 0; g4 < 4; ++g4) {
                    const f32x4 d4 = *reinterpret_cast<const f32x4*>(stat + 32 + 8 * g4 + 4 * hi);
#pragma unroll
                    for (int x = 0; x < 4; ++x) dP[s][4 * g4 + x] = d4[x];
                }
#pragma unroll
            for (int m = MP; m < 4 * MP; ++m) {
                const int step = m >> 1, s = m & 1, c = step % PH;
                const int j2 = c / (D / 32), dt = c % (D / 32);
                if (m == 2 * (4 * PH - FD)) {         // before its first fragment is read
                    // the next tile has landed (the one behind it may be in flight), and every wavefront has left the tile
                    // before this one: its stage takes the next requests
                    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((AHEAD - 1) * LOADS) : "memory");
                    if (NWK > 1) __builtin_amdgcn_s_barrier();
                    asm volatile("" ::: "memory");
                }
                if (step < 2 * PH) {
                    dP[s] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[step % FD].v, vf[s][c], dP[s], 0, 0, 0);
                } else {
                    const u32x4 bp = {pk[s][4 * j2], pk[s][4 * j2 + 1], pk[s][4 * j2 + 2], pk[s][4 * j2 + 3]};
                    if (step < 3 * PH) bw_mfma_acc(av[s][dt], fr[step % FD].v, bw_as_bf16x8(bp), dt == 0);
                    else bw_mfma_acc(ak[s][dt], fr[step % FD].v, bw_as_bf16x8(bp), dt == 0);
                }
                if (s == 1) {
                    if (step + FD == 2 * PH) BW_TR_ADDR(ta, sb)
                    if (step + FD == 4 * PH) BW_ROW_ADDR(ra, sbn)
                    BW_READ(fr[step % FD], ra, ta, (step + FD) % (4 * PH));
                }
                // half-unit u: rows 8 * (u / 4) + 4 * hi + 2 * (u % 2) + {0, 1}, key tile (u / 2) % 2
#pragma unroll
                for (int u = 0; u < 16; ++u) {
                    const int g4 = u >> 2, ks = (u >> 1) & 1, e = 4 * g4 + 2 * (u & 1);
                    if (MP + 2 + u * (3 * MP / 2 - 3) / 16 == m) {
                        if ((u & 3) == 0) {
#pragma unroll
                            for (int x = 0; x < 4; ++x) l2[x] = sr[x] * -1.4426950408889634f;
                            if (g4 < 3) sr = *reinterpret_cast<const f32x4*>(stat + 8 * g4 + 8 + 4 * hi);
                        }
#pragma unroll
                        for (int x = 0; x < 2; ++x) S[ks][e + x] = fast_exp2(fmaf(S[ks][e + x], p.scale_log2, l2[2 * (u & 1) + x]));
                        pk[ks][e >> 1] = pack_bf16x2(S[ks][e], S[ks][e + 1]);
                    }
                    if (5 * MP / 2 + u * MP / 16 == m) {
                        pk[ks][e >> 1] = pack_bf16x2(S[ks][e] * dP[ks][e], S[ks][e + 1] * dP[ks][e + 1]);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        } else {
#pragma unroll
            for (int x = 0; x <= IPW; ++x) BW_REQUEST(x);
            BW_ROW_ADDR(ra, sbn)
            asm volatile("s_waitcnt vmcnt(%0)" ::"n"((AHEAD - 1) * LOADS) : "memory");
            if (NWK > 1) __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
#pragma unroll
            for (int s = 0; s < FD; ++s) BW_READ(fr[s], ra, ta, s);
        }
        BW_ADVANCE();
        st = stn;
        rt += rt_step;
        BW_WRAP()
    }
#undef BW_WRAP
#undef BW_NEXT_HEAD
#undef BW_READ
#undef BW_ROW_ADDR
#undef BW_TR_ADDR
#undef BW_ADVANCE
#undef BW_REQUEST
#undef BW_ROW
    // the requests past the end, before the ring is reused; and the wait states between the last product and a read of its result
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_nop 15\n\ts_nop 15" ::: "memory");
    __syncthreads();

    const int le = bw_lane();                         // its offsets are formed here, not kept over the loop
    const int ne = le & 31, he = le >> 5;
    // ---- sum over the row groups, register for register --------------------------------------------------------------
    if (NWR > 1) {
        f32x4* mb = reinterpret_cast<f32x4*>(smem) + wk * (64 * D / 4) + le;
#pragma unroll
        for (int o = 0; o < 2; ++o)
            for (int src = 1; src < NWR; ++src) {
                if (wr == src) {
#pragma unroll
                    for (int x = 0; x < 2 * (D / 32) * 4; ++x) {
                        const f32x16& a = o ? ak[x / (D / 8)][x / 4 % (D / 32)] : av[x / (D / 8)][x / 4 % (D / 32)];
                        mb[x * 64] = f32x4{a[4 * (x & 3)], a[4 * (x & 3) + 1], a[4 * (x & 3) + 2], a[4 * (x & 3) + 3]};
                    }
                }
                __syncthreads();
                if (wr == 0) {
#pragma unroll
                    for (int x = 0; x < 2 * (D / 32) * 4; ++x) {
                        f32x16& a = o ? ak[x / (D / 8)][x / 4 % (D / 32)] : av[x / (D / 8)][x / 4 % (D / 32)];
                        const f32x4 v = mb[x * 64];
#pragma unroll
                        for (int e = 0; e < 4; ++e) a[4 * (x & 3) + e] += v[e];
                    }
                }
                __syncthreads();
            }
    }
    // ---- store: 32 keys at a time through a private LDS region, whole rows, 16 bytes per lane ------------------------
    if (wr == 0) {
        unsigned char* ob = smem + wk * (32 * OPB);
#pragma unroll
        for (int o = 0; o < 2; ++o)
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const float f = o ? p.scale : 1.0f;
#pragma unroll
                for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
                    for (int q4 = 0; q4 < 4; ++q4) {
                        const f32x16& a = o ? ak[s][dt] : av[s][dt];
                        u32x2 v;
                        v[0] = pack_bf16x2(a[4 * q4] * f, a[4 * q4 + 1] * f);
                        v[1] = pack_bf16x2(a[4 * q4 + 2] * f, a[4 * q4 + 3] * f);
                        *reinterpret_cast<u32x2*>(ob + ne * OPB + (32 * dt + 8 * q4 + 4 * he) * 2) = v;
                    }
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // one wavefront's LDS operations complete in order
                uint16_t* op = (o ? sdk : sdv) + kv_off + kvh * ssh;
#pragma unroll
                for (int q = 0; q < (32 * C8) / 64; ++q) {
                    const int id = q * 64 + le;
                    const int row = id / C8, c = id - row * C8;
                    const int j = jw + 32 * s + row;
                    const u32x4 v = *reinterpret_cast<const u32x4*>(ob + row * OPB + c * 16);
                    if (j < slen) *reinterpret_cast<u32x4*>(op + (int64_t)j * sst + 8 * c) = v;
                }
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
            }
    }
    __syncthreads();   // the LDS images are reused by the next pass
    }
}

// dQ with 64 rows a wavefront (two MFMA column tiles), for launches that fill the chip with such wavefronts: as in the dK / dV
// kernel every K and V fragment read from LDS then feeds two products (with 32 rows the LDS delivers no faster than the
// matrix pipes consume), and the one wavefront a SIMD holds weaves its vector work between the products: the scores of
// the NEXT key tile are formed between dP and dQ of this one, so that the exponentials run beside dP and those scores,
// and dS beside the scores and the first half of dQ.  K / V tiles come by global_load_lds through a ring of four, two tiles
// ahead.  delta = rowsum(dO * O) is formed here, from the dO fragments the kernel holds anyway, and left for the dK / dV
// kernels.
// Measured (8 x 4096 tokens, 32 / 8 heads of 128, blocks of 4): 1.53 ms = 1.09 PFLOP/s of products, 32 rows a wavefront 1.82
// ms and 0.10 for delta by itself.
template <bool BC>
__global__ __launch_bounds__(128, 1) void attn_bwd_dq64_kernel(BwdParams p, GridRemap rm) {
    constexpr int D = 128, NWQ = 2;                    // head size, wavefronts
    constexpr int NS = 4, FD = 4;
    constexpr int P = D * 2, C8 = D / 8;
    constexpr int RPI = 64 / C8, IPW = 32 / RPI / NWQ;
    constexpr int IMG = 32 / RPI * BW_GP;
    constexpr int STAGE = 2 * IMG;                     // K, V
    constexpr int LOADS = 2 * IPW;
    constexpr int OPB = D * 2 + 16;                    // output staging row pitch (bytes)
    constexpr int RING = NS * STAGE, STORE = NWQ * 32 * (OPB + 8);
    static_assert(IPW >= 1 && RING >= STORE, "ring");
    __shared__ __attribute__((aligned(1024))) unsigned char smem[RING];

    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 31, hi = lane >> 5;
    int b = blockIdx.z, kvh = blockIdx.y, bx0 = blockIdx.x;
    if (rm.nx > 0) {
        int grp;
        if (!remap_decode(rm, p.B * p.Hkv, grp, bx0)) return;
        kvh = grp % p.Hkv;
        b = grp / p.Hkv;
    }
    const int r0 = bx0 * (64 * NWQ);

    int len0 = p.seg[0].len, len1 = p.seg[1].len, len2 = p.seg[2].len;
    int R = p.R, s0 = 0;
    int64_t q_off = b * p.q_sb, o_off = b * p.o_sb, do_off = b * p.do_sb, dq_off = b * p.dq_sb, kv1_off = b * p.seg[1].sb;
    if (p.cu) {
        s0 = min(max(p.cu[b], 0), p.total);
        const int sl = max(min(min(p.cu[b + 1], p.total) - s0, p.Lq), 0);
        R = p.g * sl;
        if (r0 >= R) return;
        len1 = min(len1, sl);
        q_off = s0 * p.q_st;
        o_off = s0 * p.o_st;
        do_off = s0 * p.do_st;
        dq_off = s0 * p.dq_st;
        kv1_off = s0 * p.seg[1].st;
    }
    int F0 = 0, F1 = 0, F2 = 0, ho0 = 0, ho1 = 0, ho2 = 0;
    bool same0 = false, same1 = false, same2 = false;
    if (BC) {
        const int rows_end = min(r0 + 64 * NWQ, R);
        const int lim = ((p.q_pos0 + (rows_end - 1) / p.g) / p.bs + 1) * p.bs;
        const int first = ((p.q_pos0 + r0 / p.g) / p.bs) * p.bs;
        ho0 = (p.seg[0].rule == DLM_SEG_EARLIER_BLOCKS) ? p.bs : 0;
        ho1 = (p.seg[1].rule == DLM_SEG_EARLIER_BLOCKS) ? p.bs : 0;
        ho2 = (p.seg[2].rule == DLM_SEG_EARLIER_BLOCKS) ? p.bs : 0;
        same0 = p.seg[0].rule == DLM_SEG_SAME_BLOCK;
        same1 = p.seg[1].rule == DLM_SEG_SAME_BLOCK;
        same2 = p.seg[2].rule == DLM_SEG_SAME_BLOCK;
        len0 = max(0, min(len0, lim - ho0 - p.seg[0].pos0));
        len1 = max(0, min(len1, lim - ho1 - p.seg[1].pos0));
        len2 = max(0, min(len2, lim - ho2 - p.seg[2].pos0));
        if (same0) F0 = min(max(first - p.seg[0].pos0, 0) >> 5, (len0 + 31) >> 5);
        if (same1) F1 = min(max(first - p.seg[1].pos0, 0) >> 5, (len1 + 31) >> 5);
        if (same2) F2 = min(max(first - p.seg[2].pos0, 0) >> 5, (len2 + 31) >> 5);
    }
    const int T0 = ((len0 + 31) >> 5) - F0, T1 = ((len1 + 31) >> 5) - F1, T2 = ((len2 + 31) >> 5) - F2;
    const int T = T0 + T1 + T2;

    const uint16_t* kb0 = p.seg[0].k + b * p.seg[0].sb + kvh * p.seg[0].sh;
    const uint16_t* vb0 = p.seg[0].v + b * p.seg[0].sb + kvh * p.seg[0].sh;
    const uint16_t* kb1 = p.seg[1].k + kv1_off + kvh * p.seg[1].sh;
    const uint16_t* vb1 = p.seg[1].v + kv1_off + kvh * p.seg[1].sh;
    const uint16_t* kb2 = p.seg[2].k + b * p.seg[2].sb + kvh * p.seg[2].sh;
    const uint16_t* vb2 = p.seg[2].v + b * p.seg[2].sb + kvh * p.seg[2].sh;
    const int64_t st0 = p.seg[0].st, st1 = p.seg[1].st, st2 = p.seg[2].st;
    const int sp0 = __builtin_amdgcn_readfirstlane(p.seg[0].pos0), sp1 = __builtin_amdgcn_readfirstlane(p.seg[1].pos0),
              sp2 = __builtin_amdgcn_readfirstlane(p.seg[2].pos0);

    // ---- lane parts of the LDS addresses, as in the dK / dV kernel --------------------------------------------
    constexpr int RSH = 6, RDIV = 2;
    const int row_base = n / RPI * BW_GP + n % RPI * P + hi * 16;
    const int row_x = (n & 3) << 6;
    const int s16 = lane & 15, blk = (lane >> 4) & 1;
    const int tr_base = hi * BW_GP + (s16 >> 2) * P + ((2 * blk + ((s16 & 3) >> 1)) << 4) + 8 * (s16 & 1);
    const int tr_x = (s16 >> 2) << 6;
    const int c16 = ((lane % C8) ^ bw_swz<D>(lane / C8)) * 16;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;

    // Walk over the key tiles of all segments, twice: the tile to request (rk, rv: its first K and V row, rleft: rows from there to
    // the segment's end) and the tile to multiply (cpos: position of its first key, cleft).  Past the last tile the request
    // stays on it, for a stage nobody reads.
    int rseg = -1, rleft = 0, cseg = -1, cleft = 0, cpos = 0, choff = 0;
    bool csame = false;
    const uint16_t *rk = nullptr, *rv = nullptr;
    int64_t rst = 0;
    uint32_t voff = 0;                                // this lane's offset inside a request of the segment
#define DQ_REQ_SEG()                                                                                     \
    {                                                                                                    \
        ++rseg;                                                                                          \
        if (rseg == 0 && T0 == 0) ++rseg;                                                                \
        if (rseg == 1 && T1 == 0) ++rseg;                                                                \
        const int F_ = rseg == 0 ? F0 : (rseg == 1 ? F1 : F2);                                           \
        rst = rseg == 0 ? st0 : (rseg == 1 ? st1 : st2);                                                 \
        rk = (rseg == 0 ? kb0 : (rseg == 1 ? kb1 : kb2)) + (int64_t)(F_ * 32) * rst;                     \
        rv = (rseg == 0 ? vb0 : (rseg == 1 ? vb1 : vb2)) + (int64_t)(F_ * 32) * rst;                     \
        rleft = (rseg == 0 ? len0 : (rseg == 1 ? len1 : len2)) - F_ * 32;                                \
        voff = __umul24(lane / C8, (int)rst * 2) + c16;                                                  \
    }
    const int last_seg = T2 > 0 ? 2 : (T1 > 0 ? 1 : 0);
#define DQ_REQ_NEXT()                                                                                    \
    if (rleft > 32) {                                                                                    \
        rleft -= 32;                                                                                     \
        rk += 32 * rst;                                                                                  \
        rv += 32 * rst;                                                                                  \
    } else if (rseg != last_seg) DQ_REQ_SEG()
#define DQ_CUR_SEG()                                                                                     \
    {                                                                                                    \
        ++cseg;                                                                                          \
        if (cseg == 0 && T0 == 0) ++cseg;                                                                \
        if (cseg == 1 && T1 == 0) ++cseg;                                                                \
        const int F_ = cseg == 0 ? F0 : (cseg == 1 ? F1 : F2);                                           \
        cpos = (cseg == 0 ? sp0 : (cseg == 1 ? sp1 : sp2)) + F_ * 32;                                    \
        cleft = (cseg == 0 ? len0 : (cseg == 1 ? len1 : len2)) - F_ * 32;                                \
        choff = cseg == 0 ? ho0 : (cseg == 1 ? ho1 : ho2);                                               \
        csame = cseg == 0 ? same0 : (cseg == 1 ? same1 : same2);                                         \
    }
    // request x of the tile: rows of K and the same rows of V; rows past the segment's end repeat its last row, their scores are
    // hidden below.  (Strides of 2^24 bytes and more take 64-bit products.)
#define DQ_REQUEST(stage, x)                                                                             \
    {                                                                                                    \
        const int q_ = w * IPW + (x);                                                                    \
        const uint32_t dst_ = lds0 + (stage) * STAGE + q_ * BW_GP;                                       \
        if (rleft >= 32 && rst < (1 << 23)) {                                                            \
            bw_load_lds16_pair<IMG>(rk, rv, voff, q_ * RPI * ((int)rst * 2), dst_);                      \
        } else {                                                                                         \
            const int64_t off_ = min(q_ * RPI + lane / C8, rleft - 1) * rst + c16 / 2;                   \
            bw_load_lds16(rk + off_, dst_);                                                              \
            bw_load_lds16(rv + off_, dst_ + IMG);                                                        \
        }                                                                                                \
    }

    if (T > 0) {
        DQ_REQ_SEG()
        DQ_CUR_SEG()
#pragma unroll
        for (int t = 0; t < NS - 1; ++t) {
#pragma unroll
            for (int x = 0; x < IPW; ++x) DQ_REQUEST(t, x);
            DQ_REQ_NEXT()
        }
    }

    // ---- this lane's two query rows: Q and dO fragments (B operands), LSE and delta ---------------------------
    // Everything is requested before anything is used: one round trip, which nothing else on the SIMD covers (before: a row tile at a
    // time and its LSE behind it, four trips, 10.0 of a workgroup's 38 us on 64 k packed tokens; now 7.8, of which 3.1 are the address unit's
    // for 98 requests that touch 32 rows each).  A row past the end repeats the last one: it gets no probability and is not stored.
    bf16x8 qf[2][D / 16], dof[2][D / 16];
    float nlse2[2], ndelta[2];            // -LSE in log2 units (-inf: no probability at all), -delta
    int qlim[2];
    int qlim_min = 0x7fffffff, qlim_max = 0;
    u32x4 of[2][D / 16];
    int64_t si[2];
    float lse[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const int r = min(r0 + w * 64 + s * 32 + n, R - 1);
        const int qi = r / p.g;
        const int h = kvh * p.g + r - qi * p.g;
        const uint16_t* qp = p.q + q_off + qi * p.q_st + (int64_t)h * p.q_sh;
        const uint16_t* dp = p.dout + do_off + qi * p.do_st + (int64_t)h * p.do_sh;
        const uint16_t* op = p.o + o_off + qi * p.o_st + (int64_t)h * p.o_sh;
        si[s] = stat_index(p, b, h, qi, s0);
        lse[s] = p.lse[si[s]];
#pragma unroll
        for (int c = 0; c < D / 16; ++c) {
            qf[s][c] = bw_as_bf16x8(*reinterpret_cast<const u32x4*>(qp + 16 * c + 8 * hi));
            dof[s][c] = bw_as_bf16x8(*reinterpret_cast<const u32x4*>(dp + 16 * c + 8 * hi));
            of[s][c] = *reinterpret_cast<const u32x4*>(op + 16 * c + 8 * hi);
        }
        qlim[s] = BC ? ((p.q_pos0 + qi) / p.bs + 1) * p.bs : 0;
        if (BC) {
            qlim_min = min(qlim_min, qlim[s]);
            qlim_max = max(qlim_max, qlim[s]);
        }
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        float acc = 0.f;
#pragma unroll
        for (int c = 0; c < D / 16; ++c) {
            union { bf16x8 b; u32x4 u; } d;
            d.b = dof[s][c];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                acc += bf16_bits_to_f32(of[s][c][e] & 0xffffu) * bf16_bits_to_f32(d.u[e] & 0xffffu);
                acc += bf16_bits_to_f32(of[s][c][e] >> 16) * bf16_bits_to_f32(d.u[e] >> 16);
            }
        }
        acc += shfl_xor(acc, 32);
        ndelta[s] = -acc;
        const bool valid = r0 + w * 64 + s * 32 + n < R;
        nlse2[s] = valid && lse[s] > -INFINITY ? lse[s] * -1.4426950408889634f : -INFINITY;
        if (valid && hi == 0) p.delta[si[s]] = -acc;
    }
    if (BC) {
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
            qlim_min = min(qlim_min, shfl_xor(qlim_min, off));
            qlim_max = max(qlim_max, shfl_xor(qlim_max, off));
        }
        qlim_min = __builtin_amdgcn_readfirstlane(qlim_min);
        qlim_max = __builtin_amdgcn_readfirstlane(qlim_max);
    }

    constexpr int PH = D / 16, MP = 2 * PH;           // steps and MFMAs per product
    union Frag { s16x4 h[2]; bf16x8 v; };
    f32x16 dq[2][D / 32];
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
        for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
            for (int i = 0; i < 16; ++i) dq[s][dt][i] = 0.f;

#define DQ_ROW_ADDR(a, sb) _Pragma("unroll") for (int k = 0; k < 4; ++k) a[k] = (row_x ^ (k << RSH)) + ((sb) + row_base);
#define DQ_TR_ADDR(a, sb) _Pragma("unroll") for (int k = 0; k < D / 32; ++k) a[k] = (tr_x ^ (k << 6)) + ((sb) + tr_base);
    // fragment of step s: V rows of this tile, K rows of the next one (va, ka: row addresses), K^T of this one
#define DQ_READ(f, va, ka, ta, s)                                                                        \
    {                                                                                                    \
        const int c_ = (s) % PH;                                                                         \
        if ((s) < PH) f.v = *reinterpret_cast<const bf16x8*>(smem + va[c_ / RDIV] + (c_ % RDIV) * 32 + IMG); \
        else if ((s) < 2 * PH) f.v = *reinterpret_cast<const bf16x8*>(smem + ka[c_ / RDIV] + (c_ % RDIV) * 32); \
        else {                                                                                           \
            const int j2_ = c_ / (D / 32), dt_ = c_ % (D / 32);                                          \
            _Pragma("unroll") for (int q = 0; q < 2; ++q)                                                \
                f.h[q] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(smem + ta[dt_] + (2 * j2_ + q) * (8 / RPI) * BW_GP)); \
        }                                                                                                \
    }
    // Q, dO, O and the first tiles: a full wait, after which the compiler counts no load of its own inside the loop
    __builtin_amdgcn_s_waitcnt(0x0F70);               // vmcnt(0)
    if (T > 0) {
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        f32x16 SS[2][2];
        int va[4], ka[4], ta[D / 32];
        Frag fr[FD];
        DQ_ROW_ADDR(ka, 0)
        {   // scores of tile 0, not overlapped with anything
            Frag f;
#pragma unroll
            for (int c = 0; c < PH; ++c) {
                DQ_READ(f, va, ka, ta, PH + c)
#pragma unroll
                for (int s = 0; s < 2; ++s) {
                    if (c == 0) bw_mfma_zero(SS[0][s], f.v, qf[s][0]);
                    else SS[0][s] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.v, qf[s][c], SS[0][s], 0, 0, 0);
                }
            }
        }
        DQ_ROW_ADDR(va, 0)
#pragma unroll
        for (int s = 0; s < FD; ++s) DQ_READ(fr[s], va, ka, ta, s)
        // one tile: SS[v] holds its scores, SS[1 - v] takes the next tile's (two tiles a turn: no copies)
        for (int t0 = 0; t0 < T; t0 += 2)
#pragma unroll
        for (int v = 0; v < 2; ++v) {
            const int t = t0 + v;
            if (t >= T) break;
            const int sb = (t & (NS - 1)) * STAGE, sbn = ((t + 1) & (NS - 1)) * STAGE;
            if (cleft < 32 || (BC && (cpos + 31 >= qlim_min - choff || (csame && cpos < qlim_max - p.bs)))) {
#pragma unroll
                for (int s = 0; s < 2; ++s) {
                    int hi_r = cpos + cleft;
                    int lo_r = -(1 << 30);
                    if (BC) {
                        hi_r = min(hi_r, qlim[s] - choff);
                        if (csame) lo_r = qlim[s] - p.bs;
                    }
                    const unsigned span = (unsigned)max(hi_r - lo_r, 0);
                    const unsigned off0 = (unsigned)(cpos + 4 * hi - lo_r);
#pragma unroll
                    for (int i = 0; i < 16; ++i)
                        if (off0 + (unsigned)(8 * (i >> 2) + (i & 3)) >= span) SS[v][s][i] = -INFINITY;
                }
            }
            if (cleft > 32) {
                cleft -= 32;
                cpos += 32;
            } else if (cseg != last_seg) DQ_CUR_SEG()
            f32x16 dP[2];
            uint32_t pk[2][8];                        // dS as bf16 pairs: the B operand of the last product
            DQ_ROW_ADDR(va, sb)
#pragma unroll
            for (int m = 0; m < 3 * MP; ++m) {
                const int step = m >> 1, s = m & 1, c = step % PH;
                if (m == MP - 2 * FD) {
                    // the next tile has landed (the one behind it may be in flight), and every wavefront has left the tile
                    // before this one: its stage takes the requests below
                    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(LOADS) : "memory");
                    __builtin_amdgcn_s_barrier();
                    asm volatile("" ::: "memory");
                    DQ_ROW_ADDR(ka, sbn)
                }
                if (step < PH) {
                    if (c == 0) bw_mfma_zero(dP[s], fr[step % FD].v, dof[s][0]);
                    else dP[s] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[step % FD].v, dof[s][c], dP[s], 0, 0, 0);
                } else if (step < 2 * PH) {
                    if (c == 0) bw_mfma_zero(SS[1 - v][s], fr[step % FD].v, qf[s][0]);
                    else SS[1 - v][s] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[step % FD].v, qf[s][c], SS[1 - v][s], 0, 0, 0);
                } else {
                    const int j2 = c / (D / 32), dt = c % (D / 32);
                    const u32x4 bp = {pk[s][4 * j2], pk[s][4 * j2 + 1], pk[s][4 * j2 + 2], pk[s][4 * j2 + 3]};
                    bw_mfma_acc(dq[s][dt], fr[step % FD].v, bw_as_bf16x8(bp), dt == 0);
                }
                if (s == 1) {
                    if (step + FD == 2 * PH) DQ_TR_ADDR(ta, sb)
                    if (step + FD == 3 * PH) DQ_ROW_ADDR(va, sbn)
                    DQ_READ(fr[step % FD], va, ka, ta, (step + FD) % (3 * PH))
                }
                // half-unit u: keys 8 * (u / 4) + 4 * hi + 2 * (u % 2) + {0, 1}, row tile (u / 2) % 2
#pragma unroll
                for (int u = 0; u < 16; ++u) {
                    const int ks = (u >> 1) & 1, e = 4 * (u >> 2) + 2 * (u & 1);
                    if (u * 5 * MP / 64 == m) {
#pragma unroll
                        for (int x = 0; x < 2; ++x) SS[v][ks][e + x] = fast_exp2(fmaf(SS[v][ks][e + x], p.scale_log2, nlse2[ks]));
                    }
                    if (MP + 3 * MP / 16 + u * 5 * MP / 64 == m) {
                        pk[ks][e >> 1] = pack_bf16x2(SS[v][ks][e] * (dP[ks][e] + ndelta[ks]), SS[v][ks][e + 1] * (dP[ks][e + 1] + ndelta[ks]));
                        asm volatile("" : "+v"(pk[ks][e >> 1]));   // here, not behind the branches of the requests below
                    }
                }
                if (m >= 5 * MP / 2) {
#pragma unroll
                    for (int x = 0; x < IPW; ++x)
                        if (5 * MP / 2 + x * (MP / 2) / IPW == m) DQ_REQUEST((t + NS - 1) & (NS - 1), x);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            DQ_REQ_NEXT()
        }
    }
#undef DQ_REQ_SEG
#undef DQ_REQ_NEXT
#undef DQ_CUR_SEG
#undef DQ_REQUEST
#undef DQ_ROW_ADDR
#undef DQ_TR_ADDR
#undef DQ_READ
    // the requests past the end, before the ring is reused; and the wait states between the last product and a read of its result
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_nop 15\n\ts_nop 15" ::: "memory");
    __syncthreads();

    // dQ^T sits in the accumulators with lane = row: each wavefront transposes 32 rows at a time through a private LDS
    // region and stores whole rows, 16 bytes per lane
    unsigned char* ob = smem + w * (32 * OPB);
    int64_t* roff = reinterpret_cast<int64_t*>(smem + NWQ * 32 * OPB) + w * 32;
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const int r = r0 + w * 64 + s * 32 + n;
        const int qi = r / p.g;
        if (hi == 0) roff[n] = r < R ? qi * p.dq_st + (int64_t)(kvh * p.g + r - qi * p.g) * p.dq_sh : (int64_t)-1;
#pragma unroll
        for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
            for (int q4 = 0; q4 < 4; ++q4) {
                u32x2 v;
                v[0] = pack_bf16x2(dq[s][dt][4 * q4] * p.scale, dq[s][dt][4 * q4 + 1] * p.scale);
                v[1] = pack_bf16x2(dq[s][dt][4 * q4 + 2] * p.scale, dq[s][dt][4 * q4 + 3] * p.scale);
                *reinterpret_cast<u32x2*>(ob + n * OPB + (32 * dt + 8 * q4 + 4 * hi) * 2) = v;
            }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // one wavefront's LDS operations complete in order
#pragma unroll
        for (int q = 0; q < (32 * C8) / 64; ++q) {
            const int id = q * 64 + lane;
            const int row = id / C8, c = id - row * C8;
            const int64_t ro = roff[row];
            const u32x4 v = *reinterpret_cast<const u32x4*>(ob + row * OPB + c * 16);
            if (ro >= 0) *reinterpret_cast<u32x4*>(p.dq + dq_off + ro + 8 * c) = v;
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    }
}

template <int D, bool BC, int NWK, int NWR>
static int launch_dkv(const BwdParams& p, int s, hipStream_t st) {
    // Q and dO laid out alike, the usual case: a kernel without the other request paths (scalars kept in lanes of vector registers 46 -> 31 at d =
    // 128, 57 -> 31 - 42 at d = 64; forward and backward, 4 x 777 tokens, block diffusion, 4 heads of 64: 165 -> 148 us).  Not with d = 128 under a
    // block-causal mask, where the compiler then spills 48 vector registers.
    const bool alike = !(D == 128 && BC) && small_strides(p) && p.q_st == p.do_st && p.q_sh == p.do_sh;
    const int n_slabs = (p.seg[s].len + 64 * NWK - 1) / (64 * NWK);
    // equal-work pairing where the mask makes slabs unequal (not for "own block only": every slab sees one block's rows) and
    // half as many workgroups still fill the chip
    const int pair = (dkv_pairs<BC, NWK, NWR>() && p.seg[s].rule != DLM_SEG_SAME_BLOCK && n_slabs >= 4 && (int64_t)n_slabs * p.B * p.Hkv >= 1024) ? 1 : 0;
    dim3 grid(pair ? (n_slabs + 1) / 2 : n_slabs, p.Hkv, p.B);
    GridRemap rm = no_remap();
    if ((g_attn_remap & 4) && grid.x >= 2) {
        const int64_t n_wg = set_remap(rm, (int64_t)p.B * p.Hkv, (int)grid.x, false);
        if (n_wg > 0) grid = dim3((unsigned)n_wg);
        else rm = no_remap();
    }
    if (alike) hipLaunchKernelGGL((attn_bwd_dkv_kernel<D, BC, NWK, NWR, !(D == 128 && BC)>), grid, dim3(64 * NWK * NWR), 0, st, p, s, n_slabs, pair, rm);
    else hipLaunchKernelGGL((attn_bwd_dkv_kernel<D, BC, NWK, NWR, false>), grid, dim3(64 * NWK * NWR), 0, st, p, s, n_slabs, pair, rm);
    return check_hip(hipGetLastError(), "attn_bwd_dkv_kernel launch");
}

template <int D, bool BC>
static int launch_bwd(const BwdParams& p, hipStream_t st) {
    constexpr int RPB = 256 / (D / 8);
    int rc;
    dim3 grid((p.R + 127) / 128, p.Hkv, p.B);
    // 64 rows a wavefront (d = 128): one wavefront a SIMD, so only where its workgroups of two fill the 512 places twice; below
    // that the 32-row kernel's twice as many wavefronts are as fast or faster.  Whole backward pass, us, 32 / 64 rows: 1024
    // workgroups 1671 / 1556 (4096 tokens, 32 heads, blocks of 4), 2112 328 / 313, 640 87 / 87, 128 365 / 372; at d = 64 the
    // 32-row kernel leads throughout (253 / 266, 108 / 115).  And only where the rows see enough keys: nothing covers the start and
    // end of a workgroup that has its SIMDs to itself.  dQ and delta alone, 2048 workgroups, all keys seen: 73 keys 57 / 68, 152 71 / 83,
    // 256 119 / 123 and 108 / 108, 4096 workgroups with 256 keys 239 / 234, 512 331 / 311; under a block-causal mask, where half of
    // the keys are seen, 152 keys 73 / 87, 256 117 / 126, 512 306 / 301.
    int64_t keys = 0;
    for (int s = 0; s < 3; ++s)
        if (p.seg[s].rule != DLM_SEG_SAME_BLOCK) keys += p.seg[s].len;
    const bool wide = p.dq && D == 128 && (int64_t)grid.x * grid.y * grid.z >= 1024 && keys >= (BC ? 384 : 256);
    if (!wide) {
        const int rows = p.Lq * p.Hq;
        hipLaunchKernelGGL((attn_bwd_delta_kernel<D>), dim3((rows + RPB - 1) / RPB, 1, p.B), dim3(256), 0, st, p);
        if ((rc = check_hip(hipGetLastError(), "attn_bwd_delta_kernel launch")) != DLM_OK) return rc;
    }
    if (p.dq) {
        GridRemap rm = no_remap();
        if ((g_attn_remap & 1) && grid.x >= 2) {
            const int64_t n_wg = set_remap(rm, (int64_t)p.B * p.Hkv, (int)grid.x, BC && (g_attn_remap & 2));
            if (n_wg > 0) grid = dim3((unsigned)n_wg);
            else rm = no_remap();
        }
        if (wide) hipLaunchKernelGGL((attn_bwd_dq64_kernel<BC>), grid, dim3(128), 0, st, p, rm);
        else hipLaunchKernelGGL((attn_bwd_dq_kernel<D, BC>), grid, dim3(256), 0, st, p, rm);
        if ((rc = check_hip(hipGetLastError(), "attn_bwd dQ kernel launch")) != DLM_OK) return rc;
    }
    for (int s = 0; s < 3; ++s) {
        if (!p.seg[s].dk || p.seg[s].len == 0) continue;
        // Key-split: two wavefronts of 64 keys, 512 such workgroups at a time.  With at most half of them, or with up to twice
        // as many that each walk many rows (sequences of unequal length, a causal mask: the longest decide), four wavefronts
        // share a slab's row tiles instead, for a sum through LDS at the end, which few rows do not earn back, the fewer the
        // more workgroups take turns on a CU.  Whole backward pass, us, key- / row-split: 256 workgroups 4757 / 3097, 64 721 / 327;
        // 320 with 4200 rows 328 / 244, 640 with 4800 426 / 366, with 600 rows 87 / 103; 1024 with 4096 rows 1671 / 1757.  dK and dV
        // alone, d = 64 and d = 128: 32 workgroups with 60 rows 10.9 / 15.8 and 14.8 / 18.9, 292 rows 20.8 / 20.1 and 29.5 / 27.9; 256
        // with 292 rows 25.4 / 40.5 and 38.8 / 38.8, 512 rows 35.0 / 46.0 and 53.7 / 49.1, 1024 rows 52.8 / 55.7 and 77.5 / 63.4.
        const int64_t n_wg = (int64_t)((p.seg[s].len + 127) / 128) * p.Hkv * p.B;
        const bool split = n_wg < 1024 && p.R >= (n_wg <= 128 ? 256 : n_wg <= 256 ? 512 : 2048);
        // One wavefront a workgroup where a second one would have no keys: four such workgroups fit a CU, at d = 128 with a ring of
        // two tiles, which is slower over many tiles while two wavefronts a workgroup fit the chip at once.  dK and dV alone, us, two /
        // one: 4096 workgroups with 8 keys and rows 56 / 36 (d = 64) and 86 / 48 (d = 128), 64 keys and 448 rows 293 / 236 and 489 /
        // 426; 512 with 64 keys and 448 rows, d = 128, 63 / 65.
        const bool one = p.seg[s].len <= 64 && (D == 64 || n_wg > 512 || p.R <= 128);
        if (!split && one) rc = launch_dkv<D, BC, 1, 1>(p, s, st);
        else if (!split) rc = launch_dkv<D, BC, 2, 1>(p, s, st);
        else if constexpr (D == 64) rc = launch_dkv<D, BC, 1, 4>(p, s, st);
        else rc = launch_dkv<D, BC, 2, 2>(p, s, st);
        if (rc != DLM_OK) return rc;
    }
    return DLM_OK;
}

static int validate_bwd_seg(const dlm_kv_seg& s, const void* dk, const void* dv, const char* name, int d) {
    if (s.len < 0) return fail(DLM_ERR_INVALID_ARG, "block_attn_bwd: %s.len < 0", name);
    if (s.rule < DLM_SEG_CAUSAL || s.rule > DLM_SEG_SAME_BLOCK) return fail(DLM_ERR_INVALID_ARG, "block_attn_bwd: %s.rule %d unknown", name, s.rule);
    if ((dk == nullptr) != (dv == nullptr)) return fail(DLM_ERR_INVALID_ARG, "block_attn_bwd: d%s k and v gradients go together", name);
    if (s.len == 0) return DLM_OK;
    if (!s.k || !s.v) return fail(DLM_ERR_INVALID_ARG, "block_attn_bwd: %s has null k/v", name);
    if (!aligned16(s.k) || !aligned16(s.v) || !aligned16(dk) || !aligned16(dv))
        return fail(DLM_ERR_UNSUPPORTED, "block_attn_bwd: %s pointers not 16-byte aligned", name);
    if ((s.stride_b | s.stride_h | s.stride_t) % 8) return fail(DLM_ERR_UNSUPPORTED, "block_attn_bwd: %s strides must be multiples of 8", name);
    if (s.stride_t < d) return fail(DLM_ERR_INVALID_ARG, "block_attn_bwd: %s.stride_t < d", name);
    if (s.pos0 < 0 || (int64_t)s.pos0 + s.len > (1 << 30)) return fail(DLM_ERR_INVALID_ARG, "block_attn_bwd: %s positions outside [0, 2^30]", name);
    return DLM_OK;
}

static int validate_bwd(const dlm_attn_bwd_args* a) {
    if (!a) return fail(DLM_ERR_INVALID_ARG, "block_attn_bwd: null args");
    if (a->struct_size != sizeof(dlm_attn_bwd_args))
        return fail(DLM_ERR_INVALID_ARG, "block_attn_bwd: struct_size %u != %zu", a->struct_size, sizeof(dlm_attn_bwd_args));
    if (a->B < 0 || a->Lq < 0 || a->Hq <= 0 || a->Hkv <= 0 || a->d <= 0)
        return fail(DLM_ERR_INVALID_ARG, "block_attn_bwd: bad sizes B=%d Lq=%d Hq=%d Hkv=%d d=%d", a->B, a->Lq, a->Hq, a->Hkv, a->d);
    if (a->Hq % a->Hkv) return fail(DLM_ERR_INVALID_ARG, "block_attn_bwd: Hq=%d is not a multiple of Hkv=%d", a->Hq, a->Hkv);
    if (a->d != 64 && a->d != 128) return fail(DLM_ERR_UNSUPPORTED, "block_attn_bwd: head_dim %d (supported: 64, 128)", a->d);
    if (a->mask_mode != DLM_MASK_FULL && a->mask_mode != DLM_MASK_BLOCK_CAUSAL)
        return fail(DLM_ERR_INVALID_ARG, "block_attn_bwd: unknown mask_mode %d", a->mask_mode);
    if (a->mask_mode == DLM_MASK_FULL && (a->prefix.rule | a->block.rule | a->suffix.rule))
        return fail(DLM_ERR_INVALID_ARG, "block_attn_bwd: segment rules need the block-causal mask mode");
    if (a->mask_mode == DLM_MASK_BLOCK_CAUSAL) {
        if (a->block_size < 1) return fail(DLM_ERR_INVALID_ARG, "block_attn_bwd: block-causal needs block_size >= 1");
        if (a->q_pos0 < 0 || (int64_t)a->q_pos0 + a->Lq + a->block_size > (1 << 30))
            return fail(DLM_ERR_INVALID_ARG, "block_attn_bwd: query positions outside [0, 2^30]");
    }
    if (a->B > 65535 || a->Hkv > 65535) return fail(DLM_ERR_UNSUPPORTED, "block_attn_bwd: B or Hkv above 65535");
    if ((int64_t)a->Lq * (a->Hq / a->Hkv) > (1 << 30)) return fail(DLM_ERR_UNSUPPORTED, "block_attn_bwd: too many rows per KV head");
    if (a->cu_seqlens) {
        if (a->prefix.len || a->suffix.len) return fail(DLM_ERR_INVALID_ARG, "block_attn_bwd: packed mode takes the block segment only");
        if (a->block.len != a->Lq) return fail(DLM_ERR_INVALID_ARG, "block_attn_bwd: packed mode needs block.len == Lq");
        if (a->total_tokens < 0 || (int64_t)a->total_tokens > (int64_t)a->B * a->Lq)
            return fail(DLM_ERR_INVALID_ARG, "block_attn_bwd: total_tokens outside [0, B * Lq]");
        if (a->total_tokens == 0) return DLM_OK;
    }
    int rc;
    if ((rc = validate_bwd_seg(a->prefix, a->d_prefix_k, a->d_prefix_v, "prefix", a->d)) != DLM_OK) return rc;
    if ((rc = validate_bwd_seg(a->block, a->d_block_k, a->d_block_v, "block", a->d)) != DLM_OK) return rc;
    if ((rc = validate_bwd_seg(a->suffix, a->d_suffix_k, a->d_suffix_v, "suffix", a->d)) != DLM_OK) return rc;
    if ((int64_t)a->prefix.len + a->block.len + a->suffix.len > (1 << 30))
        return fail(DLM_ERR_UNSUPPORTED, "block_attn_bwd: more than 2^30 keys");
    if (a->B == 0 || a->Lq == 0) return DLM_OK;
    if (!a->q || !a->out || !a->d_out || !a->lse) return fail(DLM_ERR_INVALID_ARG, "block_attn_bwd: null q/out/d_out/lse");
    if (!aligned16(a->q) || !aligned16(a->out) || !aligned16(a->d_out) || !aligned16(a->d_q))
        return fail(DLM_ERR_UNSUPPORTED, "block_attn_bwd: q/out/d_out/d_q not 16-byte aligned");
    if ((a->q_stride_b | a->q_stride_t | a->q_stride_h | a->o_stride_b | a->o_stride_t | a->o_stride_h |
         a->do_stride_b | a->do_stride_t | a->do_stride_h | a->dq_stride_b | a->dq_stride_t | a->dq_stride_h) % 8)
        return fail(DLM_ERR_UNSUPPORTED, "block_attn_bwd: strides must be multiples of 8");
    if (a->q_stride_h < a->d || a->o_stride_h < a->d || a->do_stride_h < a->d || (a->d_q && a->dq_stride_h < a->d))
        return fail(DLM_ERR_INVALID_ARG, "block_attn_bwd: head stride < d");
    if (!(a->scale == a->scale)) return fail(DLM_ERR_INVALID_ARG, "block_attn_bwd: scale is NaN");
    return DLM_OK;
}

}  // namespace dlm

using namespace dlm;

extern "C" size_t dlm_block_attn_bwd_workspace_bytes(const dlm_attn_bwd_args* a) {
    if (!a || a->B <= 0 || a->Lq <= 0 || a->Hq <= 0) return 0;
    const size_t rows = a->cu_seqlens ? (size_t)(a->total_tokens > 0 ? a->total_tokens : 0) : (size_t)a->B * a->Lq;
    return rows * (size_t)a->Hq * sizeof(float);
}

extern "C" int dlm_block_attn_bwd(const dlm_attn_bwd_args* a, void* stream) {
    int rc = validate_bwd(a);
    if (rc != DLM_OK) return rc;
    if (a->B == 0 || a->Lq == 0 || (a->cu_seqlens && a->total_tokens == 0)) return DLM_OK;
    const size_t need = dlm_block_attn_bwd_workspace_bytes(a);
    if (!a->workspace || a->workspace_bytes < need)
        return fail(DLM_ERR_WORKSPACE, "block_attn_bwd: workspace of %zu bytes needed, %zu given", need, a->workspace ? a->workspace_bytes : (size_t)0);
    if (!aligned16(a->workspace)) return fail(DLM_ERR_WORKSPACE, "block_attn_bwd: workspace not 16-byte aligned");
    BwdParams p;
    p.B = a->B; p.Lq = a->Lq; p.Hq = a->Hq; p.Hkv = a->Hkv; p.g = a->Hq / a->Hkv; p.R = p.g * a->Lq;
    p.q = (const uint16_t*)a->q; p.o = (const uint16_t*)a->out; p.dout = (const uint16_t*)a->d_out;
    p.q_sb = a->q_stride_b; p.q_st = a->q_stride_t; p.q_sh = a->q_stride_h;
    p.o_sb = a->o_stride_b; p.o_st = a->o_stride_t; p.o_sh = a->o_stride_h;
    p.do_sb = a->do_stride_b; p.do_st = a->do_stride_t; p.do_sh = a->do_stride_h;
    p.dq = (uint16_t*)a->d_q; p.dq_sb = a->dq_stride_b; p.dq_st = a->dq_stride_t; p.dq_sh = a->dq_stride_h;
    const dlm_kv_seg* segs[3] = {&a->prefix, &a->block, &a->suffix};
    void* dks[3] = {a->d_prefix_k, a->d_block_k, a->d_suffix_k};
    void* dvs[3] = {a->d_prefix_v, a->d_block_v, a->d_suffix_v};
    for (int s = 0; s < 3; ++s) {
        p.seg[s].k = (const uint16_t*)segs[s]->k; p.seg[s].v = (const uint16_t*)segs[s]->v;
        p.seg[s].dk = (uint16_t*)dks[s]; p.seg[s].dv = (uint16_t*)dvs[s];
        p.seg[s].len = segs[s]->len; p.seg[s].pos0 = segs[s]->pos0;
        p.seg[s].sb = segs[s]->stride_b; p.seg[s].sh = segs[s]->stride_h; p.seg[s].st = segs[s]->stride_t;
        p.seg[s].rule = segs[s]->rule;
    }
    p.lse = a->lse; p.delta = (float*)a->workspace;
    p.bs = a->block_size; p.q_pos0 = a->q_pos0;
    p.scale = a->scale > 0.f ? a->scale : 1.0f / sqrtf((float)a->d);
    p.scale_log2 = p.scale * 1.4426950408889634f;
    p.cu = a->cu_seqlens; p.total = a->total_tokens;
    hipStream_t st = (hipStream_t)stream;
    const bool bc = a->mask_mode == DLM_MASK_BLOCK_CAUSAL;
    if (a->d == 128) return bc ? launch_bwd<128, true>(p, st) : launch_bwd<128, false>(p, st);
    return bc ? launch_bwd<64, true>(p, st) : launch_bwd<64, false>(p, st);
}
