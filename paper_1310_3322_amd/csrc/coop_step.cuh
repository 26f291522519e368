// Cooperative tile step for large state counts (NP = 16 R).
//
// One workgroup of R / BO waves advances one tile of 16 sequences of one
// model.  Wave w owns the BO 16-state output blocks r = BO w .. BO w + BO - 1:
// it keeps the MFMA A operand of A_k^T for those blocks (4 R BO registers per
// lane) and computes, for each owned block,
//   u[s][16 r + j] = sum_i alphahat[s][i] A_k[i][16 r + j]
// as 4 R chained 16x16x4 FP32 MFMAs whose B operand (all NP states of
// alphahat, loaded once for the BO chains) comes from the workgroup's
// exchange buffer in LDS.  Each step
// every wave writes its block of alpha~ = u o b and its block's share of the
// per-sequence sum; after one barrier every wave reads all blocks and all
// shares, forms c_t and its exponent e_t (identically in every wave, fixed
// summation order) while the next step's product runs on the unscaled alpha~,
// and scales the product by 2^-e_t.
//
// Lane layout inside a wave is the one of the 16x16x4 result tile: lane l
// holds sequence l % 16 and the four states 16 r + 4 (l / 16) + 0..3 of each
// owned block r.
#pragma once

#include "common.cuh"
#include "split3.cuh"

namespace hmm {

template <int R>
struct CoopShape {
    static constexpr int NP = 16 * R;
    static constexpr int XROW = NP + 4;   // padded row of the exchange buffer (floats)
    // exchange buffer: [2][16][XROW] alpha~, then [2][R][16] block sums
    static constexpr int x_floats = 2 * TILE * XROW;
    static constexpr int p_floats = 2 * R * TILE;
    static constexpr int floats = x_floats + p_floats;
};

// A operand fragments of owned block r0 + b:
// af[b][rp][v] = A_k[16 rp + 4 g + v][16 (r0 + b) + sl].
template <int R, int BO>
__device__ __forceinline__ void coop_load_fwd_fragments(float (&af)[BO][R][4], const float *Ak, int N, int r0, int g,
                                                        int sl) {
    const int lane_off = opaque(4 * g * N + 16 * r0 + sl);
#pragma unroll
    for (int b = 0; b < BO; ++b)
#pragma unroll
        for (int rp = 0; rp < R; ++rp)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int i = 16 * rp + 4 * g + v, j = 16 * (r0 + b) + sl;
                af[b][rp][v] = (i < N && j < N) ? Ak[lane_off + (16 * rp + v) * N + 16 * b] : 0.0f;
            }
}

// A operand fragments of A_k itself for beta = A w:
// ab[b][rp][v] = A_k[16 (r0 + b) + sl][16 rp + 4 g + v].
template <int R, int BO>
__device__ __forceinline__ void coop_load_bwd_fragments(float (&ab)[BO][R][4], const float *Ak, int N, int r0, int g,
                                                        int sl) {
    const int lane_off = opaque((16 * r0 + sl) * N + 4 * g);
#pragma unroll
    for (int b = 0; b < BO; ++b)
#pragma unroll
        for (int rp = 0; rp < R; ++rp)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int i = 16 * (r0 + b) + sl, j = 16 * rp + 4 * g + v;
                ab[b][rp][v] = (i < N && j < N) ? Ak[lane_off + 16 * b * N + 16 * rp + v] : 0.0f;
            }
}

// Per-sequence sum of the previous step from the block shares (fixed order).
template <int R>
__device__ __forceinline__ float coop_step_sum(const float *psum, int sl) {
    float cs = 0.0f;
#pragma unroll
    for (int w = 0; w < R; ++w) cs = cs + psum[w * TILE + sl];
    return cs;
}

// u[b] = (frag-matrix[b] . X) 2^-e over all NP states for each owned block b, X
// read from the exchange buffer rows (layout [16][XROW]).  Scaling the product
// rather than its operand gives the same values (a power of two commutes with
// FP32 rounding away from the subnormal range), takes 4 BO ldexps per lane
// instead of 4 R, and lets the chain start before e is known.  Each chain is a
// single accumulator in block order; the operands of block rp + 1 are loaded
// while the MFMAs of block rp issue, and scheduling barriers keep the compiler
// from hoisting every load.
// q0 is the lane's first float4 of the row (block rp = 0), which a caller may
// request before it forms e (the two LDS reads then overlap).
template <int R, int BO>
__device__ __forceinline__ void coop_matvec_q0(const float (&f)[BO][R][4], const float *xrow_base, float4 q0, int e,
                                               int g, int sl, floatx4 (&u)[BO]) {
#pragma unroll
    for (int b = 0; b < BO; ++b) u[b] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
    const float *row = xrow_base + sl * CoopShape<R>::XROW + 4 * g;
    float4 qn = q0;
#pragma unroll
    for (int rp = 0; rp < R; ++rp) {
        const float4 q = qn;
        if (rp + 1 < R) qn = *(const float4 *)&row[16 * (rp + 1)];
        const float in[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
            for (int b = 0; b < BO; ++b) u[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(f[b][rp][v], in[v], u[b], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int b = 0; b < BO; ++b)
#pragma unroll
        for (int v = 0; v < 4; ++v) u[b][v] = ldexp_f(u[b][v], -e);
}

template <int R, int BO>
__device__ __forceinline__ void coop_matvec(const float (&f)[BO][R][4], const float *xrow_base, int e, int g, int sl,
                                            floatx4 (&u)[BO]) {
    const float4 q0 = *(const float4 *)&xrow_base[sl * CoopShape<R>::XROW + 4 * g];
    coop_matvec_q0<R, BO>(f, xrow_base, q0, e, g, sl, u);
}

// Fragments streamed from memory instead of registers, for state counts whose fragments
// and count accumulators do not fit the register file together: a wave's are [R blocks
// rp][BO][64 lanes] float4 (v = 0..3 in the float4), one scalar pointer runs through
// them with the loads of a block at immediate offsets (one offset register per load
// would live across the step loop), and D blocks are in flight.  Loads return in order,
// so whatever a kernel requests from memory before a product delays its fragments by that
// request's latency; prime() requests the first D blocks and may be placed ahead of
// the barrier that publishes X.  Same chains and order as coop_matvec, so the results are
// bit-identical to it.
template <int R, int BO, int D>
struct CoopStream {
    typedef const __attribute__((address_space(1))) char *gptr;  // (a generic pointer makes the loads flat)
    gptr next;
    floatx4 ring[D][BO];
    __device__ __forceinline__ void fetch(floatx4 (&f)[BO], int lane) {
        const uint32_t l16 = (uint32_t)lane * 16u;
        asm volatile("" : "+s"(next));
#pragma unroll
        for (int b = 0; b < BO; ++b)
            f[b] = *(const __attribute__((address_space(1))) floatx4 *)(next + l16 + b * (WAVE * 16));
        next += BO * WAVE * 16;
    }
    __device__ __forceinline__ void prime(const float4 *fr, int lane) {
        const uint64_t p = (uint64_t)fr;  // wave-uniform
        const uint32_t lo = __builtin_amdgcn_readfirstlane((int)(uint32_t)p), hi = __builtin_amdgcn_readfirstlane((int)(p >> 32));
        next = (gptr)(((uint64_t)hi << 32) | lo);
#pragma unroll
        for (int dd = 0; dd < D; ++dd) fetch(ring[dd], lane);
    }
    // after prime(); q0 as in coop_matvec_q0
    __device__ __forceinline__ void matvec(const float *xrow_base, float4 q0, int e, int lane, floatx4 (&u)[BO]) {
        const float *row = xrow_base + (lane & 15) * CoopShape<R>::XROW + 4 * (lane >> 4);
#pragma unroll
        for (int b = 0; b < BO; ++b) u[b] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
        float4 qn = q0;
#pragma unroll
        for (int rp = 0; rp < R; ++rp) {
            const float in[4] = {qn.x, qn.y, qn.z, qn.w};
            if (rp + 1 < R) qn = *(const float4 *)&row[16 * (rp + 1)];
#pragma unroll
            for (int v = 0; v < 4; ++v)
#pragma unroll
                for (int b = 0; b < BO; ++b)
                    u[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(ring[rp % D][b][v], in[v], u[b], 0, 0, 0);
            if (rp + D < R) fetch(ring[rp % D], lane);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int b = 0; b < BO; ++b)
#pragma unroll
            for (int v = 0; v < 4; ++v) u[b][v] = ldexp_f(u[b][v], -e);
    }
};

// alpha~ block = u o b, its share of the per-sequence sum (identical in the 4
// lanes of a sequence).
__device__ __forceinline__ float coop_emit(const floatx4 &u, const float4 &b, float (&x)[4]) {
#pragma clang fp contract(off)
    x[0] = u[0] * b.x;
    x[1] = u[1] * b.y;
    x[2] = u[2] * b.z;
    x[3] = u[3] * b.w;
    const float part = ((x[0] + x[1]) + x[2]) + x[3];
    return sum_row_groups(part);
}

// ---- The same step on the bf16 matrix cores (split3.cuh).
//
// alpha~ is exchanged as its three bf16 pieces, written once by the wave that forms
// it: piece p of sequence s is a row of NP values in chunks of 16 bytes, chunk
// (c, g) holding the states 32 c + 4 g + 0..3 and 32 c + 16 + 4 g + 0..3, which is
// the B operand of lane (s, g) for the K = 32 block c (one 16-byte LDS read).  Rows
// are padded by 16 bytes, so that the 16 lanes of an LDS pass hit 16 bank groups.
//
// Two accumulators per output block: the products hi hi, and the five smaller ones,
// added at the end, so that the small terms are not rounded into the large sum block
// by block and two chains fill the matrix core's latency.
template <int R>
struct SplitShape {
    static constexpr int NP = 16 * R;
    static constexpr int ROW = NP * 2 + 16;      // bytes of one sequence's row of a piece
    static constexpr int PIECE = TILE * ROW;
    static constexpr int BUF = 3 * PIECE;        // one step's exchange
    // shares of the per-sequence sum: one per group of GS blocks, rows of PSR floats
    // (padded to 4, the padding zero) per sequence
    static constexpr int GS = R > 8 ? 2 : 1;
    static constexpr int NG = R / GS;
    static constexpr int PSR = (NG + 3) / 4 * 4 + 4;
    static constexpr int PS = TILE * PSR;
};

// Fragments of owned blocks r0 + b: slot j of a[b][c] is A[i][o] (A^T rows, forward) with
// o = 16 (r0 + b) + sl and i = 32 c + 16 (j / 4) + 4 g + j % 4.
template <int R, int BO>
struct SplitFrags {
    Split8 a[BO][R / 2];
    __device__ __forceinline__ void load_fwd(const SplitConst &sc, const float *Ak, int N, int r0, int g, int sl) {
        const int lane_off = opaque(4 * g * N + 16 * r0 + sl);
#pragma unroll
        for (int b = 0; b < BO; ++b)
#pragma unroll
            for (int c = 0; c < R / 2; ++c) {
                float q[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const int i0 = 32 * c + 16 * (j / 4) + j % 4;
                    q[j] = (i0 + 4 * g < N && 16 * (r0 + b) + sl < N) ? Ak[lane_off + i0 * N + 16 * b] : 0.0f;
                }
                // (kept out of the branches around the loads, where each would wait for its load)
#pragma unroll
                for (int j = 0; j < 8; ++j) q[j] = ldexp_f(__int_as_float(opaque(__float_as_int(q[j]))), SPLIT_SHIFT);
                a[b][c] = split8(sc, q);
                // Four blocks take the register file of a SIMD: 21 of the 32 fragments (252
                // registers) are put into accumulation registers here, where the matrix
                // instructions read them; left to itself the compiler copied 223 registers
                // back on every step (forward of 256 states, 16384 sequences: 22.2 -> 19.9 ms).
                if constexpr (BO == 4) {
                    if (b * (R / 2) + c < 21) {
#pragma unroll
                        for (int p = 0; p < 3; ++p) {
                            uintx4 w = __builtin_bit_cast(uintx4, a[b][c].p[p]);
                            asm volatile("" : "+a"(w));
                            a[b][c].p[p] = __builtin_bit_cast(bf16x8, w);
                        }
                    }
                }
            }
    }
};

// Chunk (c, g) of sequence sl in every piece.
template <int R>
__device__ __forceinline__ void split_read(const unsigned char *buf, int c, int g, int sl, bf16x8 (&q)[3]) {
    using SH = SplitShape<R>;
#pragma unroll
    for (int p = 0; p < 3; ++p) q[p] = *(const bf16x8 *)(buf + p * SH::PIECE + sl * SH::ROW + 64 * c + 16 * g);
}

// u[b] = (fragments . X) 2^-e, X from the exchange buffer, e the exponent of X's sum (the
// fragments' 2^SPLIT_SHIFT stays in u, X's goes with its sum); q0: its chunk 0, which a caller
// may request before it forms e.  The operands of chunk c + 1 are read while chunk c's
// products issue; the scheduling barriers keep the compiler from hoisting every read.
template <int R, int BO>
__device__ __forceinline__ void split_matvec(const SplitFrags<R, BO> &f, const unsigned char *buf, const bf16x8 (&q0)[3],
                                             int e, int g, int sl, floatx4 (&u)[BO]) {
    floatx4 lo[BO];
#pragma unroll
    for (int b = 0; b < BO; ++b) u[b] = lo[b] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
    bf16x8 qn[3] = {q0[0], q0[1], q0[2]};
#pragma unroll
    for (int c = 0; c < R / 2; ++c) {
        const bf16x8 q[3] = {qn[0], qn[1], qn[2]};
        if (c + 1 < R / 2) split_read<R>(buf, c + 1, g, sl, qn);
#pragma unroll
        for (int t = 0; t < SPLIT_TERMS; ++t)
#pragma unroll
            for (int b = 0; b < BO; ++b) {
                floatx4 &acc = t == SPLIT_TERMS - 1 ? u[b] : lo[b];
                acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f.a[b][c].p[SPLIT_A[t]], q[SPLIT_X[t]], acc, 0, 0, 0);
            }
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int b = 0; b < BO; ++b)
#pragma unroll
        for (int v = 0; v < 4; ++v) u[b][v] = ldexp_f(u[b][v] + lo[b][v], -e);
}

// Own blocks r0 .. r0 + BO - 1 of sequence sl into the exchange buffer, split.
template <int R, int BO>
__device__ __forceinline__ void split_write(const SplitConst &sc, const float (&x)[BO][4], unsigned char *buf, int r0,
                                            int g, int sl) {
    using SH = SplitShape<R>;
    unsigned char *row = buf + sl * SH::ROW + 64 * (r0 / 2) + 16 * g + 8 * (r0 & 1);
    uint32_t w[3][BO][2];
#pragma unroll
    for (int b = 0; b < BO; ++b)
#pragma unroll
        for (int h = 0; h < 2; ++h) split_pair(sc, x[b][2 * h], x[b][2 * h + 1], w[0][b][h], w[1][b][h], w[2][b][h]);
#pragma unroll
    for (int p = 0; p < 3; ++p) {
        if constexpr (BO == 1) {
            *(uint2 *)(row + p * SH::PIECE) = uint2{w[p][0][0], w[p][0][1]};
        } else {
#pragma unroll
            for (int b = 0; b < BO; b += 2)
                *(uint4 *)(row + p * SH::PIECE + 32 * b) = uint4{w[p][b][0], w[p][b][1], w[p][b + 1][0], w[p][b + 1][1]};
        }
    }
}

// The wave's shares of the per-sequence sum of x.
template <int R, int BO>
__device__ __forceinline__ void split_shares(const float (&x)[BO][4], float *psum, int r0, int g, int sl) {
#pragma clang fp contract(off)
    using SH = SplitShape<R>;
#pragma unroll
    for (int i = 0; i < BO; i += SH::GS) {
        float part = x[i][0];
#pragma unroll
        for (int b = i; b < i + SH::GS; ++b)
#pragma unroll
            for (int v = (b == i ? 1 : 0); v < 4; ++v) part = part + x[b][v];
        part = sum_row_groups(part);
        psum[sl * SH::PSR + (r0 + i) / SH::GS] = part;  // the four lanes of a sequence write the same value
    }
}

// alpha~ blocks x = u o b and the wave's shares of the per-sequence sum.
template <int R, int BO>
__device__ __forceinline__ void split_emit(const floatx4 (&u)[BO], const float4 (&b)[BO], float (&x)[BO][4], float *psum,
                                           int r0, int g, int sl) {
#pragma clang fp contract(off)
#pragma unroll
    for (int i = 0; i < BO; ++i) {
        x[i][0] = u[i][0] * b[i].x;
        x[i][1] = u[i][1] * b[i].y;
        x[i][2] = u[i][2] * b[i].z;
        x[i][3] = u[i][3] * b[i].w;
    }
    split_shares<R, BO>(x, psum, r0, g, sl);
}

// Per-sequence sum of the previous step from the shares (fixed order).
template <int R>
__device__ __forceinline__ float split_step_sum(const float *psum, int sl) {
    using SH = SplitShape<R>;
    float cs = 0.0f;
#pragma unroll
    for (int i = 0; i < SH::NG; i += 4) {
        const float4 q = *(const float4 *)&psum[sl * SH::PSR + i];
        cs = (((cs + q.x) + q.y) + q.z) + q.w;
    }
    return cs;
}

}  // namespace hmm
