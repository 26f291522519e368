// Backward (adjoint) kernel on FP32 MFMA (gfx950): Baum-Welch E-step counts.
//
// The paper's learning mode runs the Baum-Welch function of its HMM stage
// (Sec. 2.7).  Its E-step is the scaled backward recursion; with the forward
// pass rescaled by exact powers of two (alphahat_t = alpha_t 2^-E_t,
// m_T = sum_i alphahat_T(i)) the scaled backward variables are
//   betahat_T = 1 / m_T,   w_{t+1} = B[:, o_{t+1}] o betahat_{t+1} 2^-e_{t+1},
//   betahat_t = A w_{t+1},
// so that gamma_t = alphahat_t o betahat_t sums to one and
// xi_t(i,j) = alphahat_t(i) A(i,j) w_{t+1}(j).  Each sequence s of weight w_s adds
//   n_pi += w_s gamma_1,  n_B[:, o_t] += w_s gamma_t,  C += w_s alphahat_t (x) w_{t+1}
// and n_A = A o C at the end: the gradient of sum_s w_s log P_s w.r.t. ln pi,
// ln A and ln B.
//
// Memory: the forward kernel stored alphahat every L = ceil(sqrt(Tmax)) steps
// (Tmax the longest sequence of the 16-sequence tile).  The segments of L steps are
// taken last to first: alphahat is recomputed from the checkpoint with the forward
// kernel's own step code (bit-identical) into a segment buffer in global memory, which the
// backward recursion then walks.  Memory per sequence grows with sqrt(T).
//
// A tile of 16 sequences is a chain of dependent steps, so the work of a step is split
// over the four waves of a workgroup, one per SIMD, by what depends on what:
//   REC     recomputes segment j - 1 while the others are on segment j
//   WALK    betahat_t = A w_{t+1}, w_t = b_t o betahat_t 2^-e_t   (the chain itself)
//   XI      C += X^T W, X = w_s alphahat_t, W = w_{t+1}: transposed through LDS so
//           that the 16 sequences become the MFMA contraction axis
//   COUNTS  n_B^T[o_t][i] += w_s gamma_t(i) into the LDS partial of the workgroup
//           (of slots that share a symbol the lowest adds for all, in slot order),
//           written to the tile's slot of a slab of per-tile partials (deterministic),
//           or with 64-bit atomics to the global counts; n_pi
// WALK leaves w_{t+1} and betahat_t of CS steps in one half of an LDS ring; XI and
// COUNTS take them CS steps later from the other half, so the waves meet at one barrier
// every CS steps (and at one that orders global memory too every L, for REC's segments).
// Symbols are requested two chunks of CS steps ahead, emission rows and alphahat one chunk
// ahead.
//
// Bound by the latency of a step of WALK and REC (about the same: four dependent 16x16x4
// MFMAs of 33 cycles and some 20 dependent vector instructions at 16 states) while the
// tiles are few, by the matrix and vector instructions of the four parts once they fill
// the card.  An FP32 MFMA leaves no issue slot to its own wave's vector instructions, which
// is why the parts of a step gain from having a SIMD each.  Against one wave per tile that
// does all of it in turn, with every operand requested when needed, an EM iteration on
// 4096 sequences of 50-400 (12 models, 16 states, 64 symbols) went from 606 to 292 us, on
// 147 sequences of 20-200 (6 models, 5 states) from 361 to 183 us (some 50 us of either are
// fewer launches and a better order of the forward's tiles), and the counts of 65536
// sequences of 16-2048 (64 models, 32 states, 256 symbols) from 6.4 to 3.9 ms.
//
// Global counts are 64-bit fixed-point sums (common.cuh) and each tile's sums are
// formed in an order fixed by its data, so the counts do not depend on which
// workgroup takes which tile.
#include <algorithm>
#include <climits>

#include "common.cuh"
#include "fwd_step.cuh"
#include "kernels.h"

namespace hmm {
namespace {

__host__ __device__ inline int nb_swizzle_mask(int NP) { return (NP & (NP - 1)) == 0 ? NP - 4 : 0; }

enum Role { REC, WALK, XI, COUNTS, ROLES };

template <int R, int CS>
struct AdjShape {
    static constexpr int NP = 16 * R;
    static constexpr int XS = NP + 4;       // padded row of the transposition tiles
    static constexpr int static_bytes = 2 * CS * (TILE * XS * 4 + R * WAVE * 16) + TILE * XS * 4 + TILE * 4 +
                                        2 * CS * TILE * 4 + 64;
    // segment buffer: two halves (segment parity) of alphahat [L][R][64] float4 and
    // packed exponents [L][64]
    static constexpr int seg_step = WAVE * (4 * R + 1);  // floats per step
};

// The barrier between two segments for the waves that read the segment buffer.  REC writes the
// half of segment j again in the phase after XI and COUNTS request their last rows of it, so
// global memory is ordered here too, and no load of theirs is left in flight (they took its value
// at the end of the phase: nothing to wait for as it is compiled now).
__device__ __forceinline__ void segment_barrier() {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
}

// Waves per SIMD that the registers are kept to.
constexpr int adj_waves(int R, int CS) { return CS == 4 ? 2 : R == 1 ? 4 : R == 2 ? 3 : 2; }

template <int R, bool NBLDS, int CS>
__global__ void __launch_bounds__(ROLES * WAVE) __attribute__((amdgpu_waves_per_eu(adj_waves(R, CS), 8)))
k_adj_tile(DevPtrs d, AdjLaunch a) {
    using SH = AdjShape<R, CS>;
    constexpr int NP = SH::NP, XS = SH::XS;
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ __align__(16) float wring[2][CS][TILE * XS];     // w_{t+1} of the sequences that go on
    __shared__ __align__(16) float4 bring[2][CS][R][WAVE];      // betahat_t
    __shared__ __align__(16) float xt[TILE * XS];
    __shared__ float mlast[TILE];                               // m_T of each sequence
    __shared__ int32_t elast[2][CS][TILE];                      // exponents of a segment's last steps
    __shared__ int32_t tile_sh;
    const int lane = threadIdx.x & (WAVE - 1);
    const int role = __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
    const int sl = lane & 15, g = lane >> 4;
    const int K = a.K, N = a.N, M = a.M;
    const int swz = nb_swizzle_mask(NP);
    const int F = fixed_exponent(*a.wmax, a.S, a.max_len);
    float *nbl = (float *)smem;  // [M][NP] when NBLDS
    uint32_t *masktab = (uint32_t *)(nbl + (size_t)M * NP);  // [m2] slot masks of slot_mask
    const int m2 = (M + 1) / 2;

    float *segf = a.seg + (size_t)blockIdx.x * a.seg_stride;
    const int64_t half = a.seg_stride / 2;
    const int Lcap = (int)(half / SH::seg_step);
    auto seg_alpha = [&](int j) { return (float4 *)(segf + (j & 1) * half); };
    auto seg_e = [&](int j) { return (int32_t *)(segf + (j & 1) * half + (size_t)Lcap * WAVE * 4 * R); };

    const int G = gridDim.x;
    const int k_first = G >= K ? (int)(blockIdx.x % K) : (int)blockIdx.x;
    const int k_step = G >= K ? K : G;
    for (int k = k_first; k < K; k += k_step) {
        const int gbeg = a.gstart[k], gend = a.gstart[k + 1];
        const int ntiles = (gend - gbeg + TILE - 1) / TILE;
        if (ntiles == 0) continue;
        const float *btk = a.bt + (size_t)k * M * NP;
        unsigned long long *B64k = a.B64 + (size_t)k * M * NP;  // [M][NP] symbol-major global counts
        if (NBLDS) {
            __syncthreads();
            for (int i = threadIdx.x; i < M * NP; i += ROLES * WAVE) nbl[i] = 0.0f;
            for (int i = threadIdx.x; i < m2; i += ROLES * WAVE) masktab[i] = 0u;
        }
        const float *Ak = d.A + (size_t)k * N * N;
        float fr[R][R][4];  // fragments of A^T (REC) or A (WALK)
        if (role == REC) load_fwd_fragments<R>(fr, Ak, N, g, sl);
        if (role == WALK) load_bwd_fragments<R>(fr, Ak, N, g, sl);

        for (;;) {
            __syncthreads();
            if (threadIdx.x == 0) tile_sh = atomicAdd(&a.queue[k], 1);
            __syncthreads();
            const int tile = __builtin_amdgcn_readfirstlane(tile_sh);  // scalar exit: the loop holds barriers
            if (tile >= ntiles) break;

            const int pos = gbeg + tile * TILE + sl;
            const bool has = pos < gend;
            const int seq = has ? a.perm[pos] : 0;
            int32_t T = 0;
            int64_t off = 0;
            bool act = false;
            if (has) {
                T = d.lengths[seq];
                off = d.offsets[seq];
                const int mk = d.model_of_seq[seq];
                const bool bad = seq_bad(T, off, a.max_len, a.total) || mk < 0 || mk >= K;
                if (bad) T = 0;
                act = !bad && T > 0 && a.flag[pos] == 0;
            }
            // the checkpoint grid uses the forward kernel's tile maximum
            const int Tmax = __builtin_amdgcn_readfirstlane(wave_max_int(T));
            if (Tmax > 0) {
                int L = 1;
                while (L * L < Tmax) ++L;
                if (!dbg_in(L - 1, Lcap, HMM_DEBUG_SEGMENT)) return;  // segment buffer too short (debug build)
                const int nseg = (Tmax + L - 1) / L;
                const int nch = (L + CS - 1) / CS;  // chunks per segment
                const float wgt = act ? (a.weight ? a.weight[seq] : 1.0f) : 0.0f;
                const int32_t *sbase = T > 0 ? d.symbols + off : d.symbols;
                const int tlim = T > 0 ? T - 1 : 0;
                auto seg_len = [&](int j) { return min(L, Tmax - j * L); };
                auto load_sym = [&](int t) { return sbase[min(max(t, 0), tlim)]; };
                auto checked = [&](int o) { return ((unsigned)o < (unsigned)M) ? o : 0; };
                // A chunk of backward steps: t0, t0 - 1, .. (n of them, none or less than none where
                // the segment is shorter or there is no segment)
                struct Chunk {
                    int t0, n;
                };
                auto back_chunk = [&](int j, int s) {
                    const int n = j >= 0 && j < nseg ? seg_len(j) - s * CS : 0;
                    return Chunk{j * L + n - 1, n};
                };
                // the chunk `by` (1 or 2) after chunk s of segment j
                auto back_after = [&](int j, int s, int by) {
                    for (int i = 0; i < by; ++i) {
                        const bool wrap = s + 1 == nch;
                        j -= wrap ? 1 : 0;
                        s = wrap ? 0 : s + 1;
                    }
                    return back_chunk(j, s);
                };

                if (role == REC) {
                    // segment nseg - 1 - p in phase p; first step of the chunk `by` after chunk s of
                    // segment j
                    auto rec_after = [&](int j, int s, int by) {
                        for (int i = 0; i < by; ++i) {
                            const bool wrap = s + 1 == nch;
                            j -= wrap ? 1 : 0;
                            s = wrap ? 0 : s + 1;
                        }
                        return max(j, 0) * L + s * CS;
                    };
                    float4 bc[CS][R], bn[CS][R];
                    int oc[CS], on[CS], o2[CS];
                    float4 ckn[R] = {};  // checkpoint of the next phase's segment
                    int cken = 0;
                    auto load_ckpt = [&](int j) {
                        if (j >= 0 && j * L < T) {
                            const float *src = a.ckpt + ((size_t)pos * a.nck + j) * NP;
#pragma unroll
                            for (int r = 0; r < R; ++r) ckn[r] = *(const float4 *)&src[16 * r + 4 * g];
                            cken = a.ckexp[(size_t)pos * a.nck + j];
                        } else {
#pragma unroll
                            for (int r = 0; r < R; ++r) ckn[r] = float4{0.0f, 0.0f, 0.0f, 0.0f};
                            cken = 0;
                        }
                    };
                    load_ckpt(nseg - 1);
#pragma unroll
                    for (int u = 0; u < CS; ++u) {
                        oc[u] = checked(load_sym(rec_after(nseg - 1, 0, 0) + u));
                        on[u] = load_sym(rec_after(nseg - 1, 0, 1) + u);
                        gather_b<R>(&btk[(size_t)oc[u] * NP], g, bc[u]);
                    }
                    float acur[R][4];
                    for (int p = 0; p <= nseg; ++p) {
                        const int j = nseg - 1 - p;
                        const int LB = j >= 0 ? seg_len(j) : 0;
                        float4 *sa = seg_alpha(j);
                        int32_t *se = seg_e(j);
                        __syncthreads();  // the segment recomputed in the phase before is visible
                        for (int s = 0; s < nch; ++s) {
                            const int t2 = rec_after(j, s, 2);
#pragma unroll
                            for (int u = 0; u < CS; ++u) {
                                on[u] = checked(on[u]);
                                gather_b<R>(&btk[(size_t)on[u] * NP], g, bn[u]);
                                o2[u] = load_sym(t2 + u);
                            }
#pragma unroll
                            for (int u = 0; u < CS; ++u) {
                                const int tl = s * CS + u;
                                if (tl < LB) {
                                    const int t = j * L + tl;
                                    int e;
                                    if (tl == 0) {
#pragma unroll
                                        for (int r = 0; r < R; ++r) {
                                            acur[r][0] = ckn[r].x;
                                            acur[r][1] = ckn[r].y;
                                            acur[r][2] = ckn[r].z;
                                            acur[r][3] = ckn[r].w;
                                        }
                                        e = cken;
                                        load_ckpt(j - 1);
                                    } else {
                                        floatx4 uu[R];
                                        tile_matvec<R>(fr, acur, uu);
                                        emit_and_rescale<R>(uu, bc[u], acur, e);
                                    }
#pragma unroll
                                    for (int r = 0; r < R; ++r)
                                        sa[(size_t)(tl * R + r) * WAVE + lane] =
                                            float4{acur[r][0], acur[r][1], acur[r][2], acur[r][3]};
                                    se[(size_t)tl * WAVE + lane] = e;
                                    if (LB - 1 - tl < CS && g == 0) elast[j & 1][LB - 1 - tl][sl] = e;
                                    if (__ballot(t == T - 1) != 0) {  // m_T of the sequences that end here
                                        float part = 0.0f;
#pragma unroll
                                        for (int r = 0; r < R; ++r)
#pragma unroll
                                            for (int v = 0; v < 4; ++v) part += acur[r][v];
                                        const float m = sum_row_groups(part);
                                        if (t == T - 1) mlast[sl] = m;
                                    }
                                }
                            }
#pragma unroll
                            for (int u = 0; u < CS; ++u) {
                                oc[u] = on[u];
                                on[u] = o2[u];
#pragma unroll
                                for (int r = 0; r < R; ++r) bc[u][r] = bn[u][r];
                            }
                            lds_barrier();
                        }
                    }
                } else if (role == WALK) {
                    float wn[R][4];  // w_{t+1}
#pragma unroll
                    for (int r = 0; r < R; ++r)
#pragma unroll
                        for (int v = 0; v < 4; ++v) wn[r][v] = 0.0f;
                    float4 bc[CS][R], bn[CS][R];
                    int on[CS], o2[CS], ec[CS], en[CS];
#pragma unroll
                    for (int u = 0; u < CS; ++u) {
                        gather_b<R>(&btk[(size_t)checked(load_sym(back_chunk(nseg, 0).t0 - u)) * NP], g, bc[u]);
                        on[u] = load_sym(back_after(nseg, 0, 1).t0 - u);
                        ec[u] = 0;
                    }
                    int half_ring = 0;
                    for (int p = 0; p <= nseg; ++p) {
                        const int j = nseg - p;
                        const int LA = p > 0 ? seg_len(j) : 0;
                        const int32_t *se = seg_e(j);
                        __syncthreads();  // the segment is visible, and its exponents' half free for REC
#pragma unroll
                        for (int u = 0; u < CS; ++u) ec[u] = elast[j & 1][u][sl];
                        for (int s = 0; s < nch; ++s, half_ring ^= 1) {
                            const int t2 = back_after(j, s, 2).t0;
#pragma unroll
                            for (int u = 0; u < CS; ++u) {
                                gather_b<R>(&btk[(size_t)checked(on[u]) * NP], g, bn[u]);
                                o2[u] = load_sym(t2 - u);
                                const int tn = LA - 1 - ((s + 1) * CS + u);
                                en[u] = se[(size_t)max(tn, 0) * WAVE + lane];
                            }
#pragma unroll
                            for (int u = 0; u < CS; ++u) {
                                const int tl = LA - 1 - (s * CS + u);
                                if (tl >= 0) {
                                    const int t = j * L + tl;
                                    float *wt = wring[half_ring][u];
#pragma unroll
                                    for (int r = 0; r < R; ++r)
                                        *(float4 *)&wt[sl * XS + 16 * r + 4 * g] =
                                            float4{wn[r][0], wn[r][1], wn[r][2], wn[r][3]};
                                    floatx4 be[R];
                                    tile_matvec<R>(fr, wn, be);
                                    if (__ballot(t == T - 1) != 0) {
                                        const float inv = 1.0f / mlast[sl];
#pragma unroll
                                        for (int r = 0; r < R; ++r)
#pragma unroll
                                            for (int v = 0; v < 4; ++v) be[r][v] = t == T - 1 ? inv : be[r][v];
                                    }
#pragma unroll
                                    for (int r = 0; r < R; ++r)
                                        bring[half_ring][u][r][lane] = float4{be[r][0], be[r][1], be[r][2], be[r][3]};
                                    // w_t = b_t o betahat_t 2^-e_t; zero where the sequence has ended or
                                    // takes no part (its values may be inf / NaN)
                                    const bool live = act && t < T;
#pragma unroll
                                    for (int r = 0; r < R; ++r) {
                                        wn[r][0] = live ? ldexp_f(bc[u][r].x * be[r][0], -ec[u]) : 0.0f;
                                        wn[r][1] = live ? ldexp_f(bc[u][r].y * be[r][1], -ec[u]) : 0.0f;
                                        wn[r][2] = live ? ldexp_f(bc[u][r].z * be[r][2], -ec[u]) : 0.0f;
                                        wn[r][3] = live ? ldexp_f(bc[u][r].w * be[r][3], -ec[u]) : 0.0f;
                                    }
                                }
                            }
#pragma unroll
                            for (int u = 0; u < CS; ++u) {
                                on[u] = o2[u];
                                ec[u] = en[u];
#pragma unroll
                                for (int r = 0; r < R; ++r) bc[u][r] = bn[u][r];
                            }
                            lds_barrier();
                        }
                    }
                } else if (role == XI) {
                    // at the slot of a chunk, request its alphahat and take the chunk before
                    floatx4 C[R][R];
#pragma unroll
                    for (int ri = 0; ri < R; ++ri)
#pragma unroll
                        for (int rj = 0; rj < R; ++rj) C[ri][rj] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
                    float4 ac[CS][R], an[CS][R];
                    // C += X^T W with X = w_s alphahat_t, W = w_{t+1}, the chunk's operands first
                    auto take = [&](const Chunk &c, int hr) {
                        float xa[CS][4][R], wb[CS][4][R];
#pragma unroll
                        for (int u = 0; u < CS; ++u) {
                            const bool trans = act && u < c.n && c.t0 - u + 1 < T;
#pragma unroll
                            for (int r = 0; r < R; ++r)
                                *(float4 *)&xt[sl * XS + 16 * r + 4 * g] =
                                    float4{trans ? wgt * ac[u][r].x : 0.0f, trans ? wgt * ac[u][r].y : 0.0f,
                                           trans ? wgt * ac[u][r].z : 0.0f, trans ? wgt * ac[u][r].w : 0.0f};
                            wave_lds_sync();
#pragma unroll
                            for (int q = 0; q < 4; ++q)
#pragma unroll
                                for (int r = 0; r < R; ++r) {
                                    xa[u][q][r] = xt[(4 * q + g) * XS + 16 * r + sl];
                                    wb[u][q][r] = wring[hr][u][(4 * q + g) * XS + 16 * r + sl];
                                }
                            wave_lds_sync();
                        }
#pragma unroll
                        for (int u = 0; u < CS; ++u) {
                            if (u >= c.n) continue;  // (its ring entry holds an older step)
#pragma unroll
                            for (int q = 0; q < 4; ++q)
#pragma unroll
                                for (int ri = 0; ri < R; ++ri)
#pragma unroll
                                    for (int rj = 0; rj < R; ++rj)
                                        C[ri][rj] =
                                            __builtin_amdgcn_mfma_f32_16x16x4f32(xa[u][q][ri], wb[u][q][rj], C[ri][rj], 0, 0, 0);
                        }
                    };
                    Chunk cp{0, 0};
                    int half_ring = 0;
                    for (int p = 0; p <= nseg; ++p) {
                        const int j = nseg - p;
                        const float4 *sa = seg_alpha(j);
                        segment_barrier();
                        for (int s = 0; s < nch; ++s, half_ring ^= 1) {
                            const Chunk cn = back_chunk(j, s);
#pragma unroll
                            for (int u = 0; u < CS; ++u)
#pragma unroll
                                for (int r = 0; r < R; ++r)
                                    an[u][r] = sa[(size_t)(max(cn.n - 1 - u, 0) * R + r) * WAVE + lane];
                            if (cp.n > 0) take(cp, half_ring ^ 1);
#pragma unroll
                            for (int u = 0; u < CS; ++u)
#pragma unroll
                                for (int r = 0; r < R; ++r) ac[u][r] = an[u][r];
                            cp = cn;
                            lds_barrier();
                        }
                    }
                    if (cp.n > 0) take(cp, half_ring ^ 1);
                    // this tile's n_A = A o C (row base opaque: the flush's addresses are formed
                    // here, not kept live across the tile loop)
                    const int rb = opaque(k * N + 4 * g);
#pragma unroll
                    for (int ri = 0; ri < R; ++ri)
#pragma unroll
                        for (int rj = 0; rj < R; ++rj)
#pragma unroll
                            for (int v = 0; v < 4; ++v) {
                                const int i = 16 * ri + 4 * g + v, jj = 16 * rj + sl;
                                const size_t e = (size_t)(rb + 16 * ri + v) * N + jj;
                                if (i < N && jj < N) add_fixed(&a.A64[e], d.A[e] * C[ri][rj][v], F, &a.nanflag[k]);
                            }
                } else {
                    // COUNTS, likewise one chunk behind
                    float nan_acc = 0.0f;  // NaN once a gamma was not finite
                    int states = 0;        // bit 4 r + v: the lane's state 16 r + 4 g + v is below N
#pragma unroll
                    for (int q = 0; q < 4 * R; ++q) states |= (16 * (q / 4) + 4 * g + q % 4 < N ? 1 : 0) << q;
                    float4 ac[CS][R], an[CS][R];
                    int oc[CS], on[CS];
#pragma unroll
                    for (int u = 0; u < CS; ++u) oc[u] = 0;
                    // gamma_t = alphahat_t o betahat_t of the chunk's steps, then their counts (steps and
                    // sequences that are not live add zero)
                    auto take = [&](const Chunk &c, int hr) {
                        float gm[CS][R][4];
#pragma unroll
                        for (int u = 0; u < CS; ++u) {
                            const uint32_t live = act && u < c.n && c.t0 - u < T ? ~0u : 0u;
#pragma unroll
                            for (int r = 0; r < R; ++r) {
                                const float4 be = bring[hr][u][r][lane];
                                const float4 al = ac[u][r];
                                const float x[4] = {wgt * al.x * be.x, wgt * al.y * be.y, wgt * al.z * be.z, wgt * al.w * be.w};
#pragma unroll
                                for (int v = 0; v < 4; ++v) {
                                    const uint32_t keep = live & (uint32_t)__builtin_amdgcn_sbfe(states, 4 * r + v, 1);
                                    gm[u][r][v] = __uint_as_float(__float_as_uint(x[v]) & keep);
                                    nan_acc = fmaf(gm[u][r][v], 0.0f, nan_acc);
                                }
                            }
                        }
                        if (NBLDS) {
                            // The lowest live slot of a symbol adds for all that share it, in slot order.
                            // It finds the others' gamma where their betahat was in the ring, so that a
                            // step is one round trip to its entry; the first NEAR of them are requested
                            // for all steps at once, before the entries.  More of them cost registers and
                            // reads, fewer a round trip each: an EM iteration with one, two, three of them
                            // took 1130, 1083, 1051 us where symbols are often shared (8 states, 6 symbols,
                            // 300 sequences of 20-1500), 880, 890, 948 on 30 symbols, 261, 273, 290 on 64 (12
                            // models of 16 states, 2000 sequences of 50-400); in chunks of two 284, 296,
                            // 306 on 64 symbols (4096 sequences) and 960, 942, 918 on 6 (40000 of 50-600).
                            constexpr int NEAR = CS / 2;
                            uint32_t rest[CS];  // the other slots whose gamma this lane adds
                            bool leads[CS];
                            float4 near[CS][NEAR][R];
                            bool any = false;
                            uint32_t word[CS];
#pragma unroll
                            for (int u = 0; u < CS; ++u) word[u] = slot_mask(masktab, oc[u], sl, act && u < c.n && c.t0 - u < T);
#pragma unroll
                            for (int u = 0; u < CS; ++u) {
                                const uint32_t m = (word[u] >> ((oc[u] & 1) << 4)) & 0xffffu;
                                leads[u] = (m & ((2u << sl) - 1u)) == (1u << sl);
                                rest[u] = leads[u] ? m & (m - 1u) : 0u;
                                any |= rest[u] != 0u;
                            }
                            const bool shared = __ballot(any) != 0;
                            uint32_t later[CS];
                            if (shared) {
#pragma unroll
                                for (int u = 0; u < CS; ++u)
#pragma unroll
                                    for (int r = 0; r < R; ++r)
                                        bring[hr][u][r][lane] = float4{gm[u][r][0], gm[u][r][1], gm[u][r][2], gm[u][r][3]};
                                wave_lds_sync();
#pragma unroll
                                for (int u = 0; u < CS; ++u) {
                                    uint32_t m = rest[u];  // (m & (m - 1) is 0 for 0)
#pragma unroll
                                    for (int n = 0; n < NEAR; ++n) {
                                        const int from = m ? 16 * g + (int)__builtin_ctz(m) : lane;
#pragma unroll
                                        for (int r = 0; r < R; ++r) near[u][n][r] = bring[hr][u][r][from];
                                        m &= m - 1u;
                                    }
                                    later[u] = m;
                                }
                            }
                            auto plus = [](float4 x, float4 y) {
                                return float4{x.x + y.x, x.y + y.y, x.z + y.z, x.w + y.w};
                            };
#pragma unroll
                            for (int u = 0; u < CS; ++u) {
                                const uint32_t m = rest[u];
                                float4 x[R];
                                auto at = [&](int r) {
                                    return (float4 *)&nbl[oc[u] * NP + ((16 * r + 4 * g) ^ (oc[u] * 4 & swz))];
                                };
#pragma unroll
                                for (int r = 0; r < R; ++r) x[r] = plus(*at(r), float4{gm[u][r][0], gm[u][r][1], gm[u][r][2], gm[u][r][3]});
                                if (shared) {
                                    uint32_t q = m;
#pragma unroll
                                    for (int n = 0; n < NEAR; ++n) {
                                        if (q) {
#pragma unroll
                                            for (int r = 0; r < R; ++r) x[r] = plus(x[r], near[u][n][r]);
                                        }
                                        q &= q - 1u;
                                    }
                                    uint32_t l = later[u];
                                    while (__ballot(l != 0) != 0) {
                                        if (l) {
                                            const int from = 16 * g + (int)__builtin_ctz(l);
#pragma unroll
                                            for (int r = 0; r < R; ++r) x[r] = plus(x[r], bring[hr][u][r][from]);
                                        }
                                        l &= l - 1u;
                                    }
                                }
                                if (leads[u]) {
#pragma unroll
                                    for (int r = 0; r < R; ++r) *at(r) = x[r];
                                }
                                wave_lds_sync();
                            }
                        } else {
#pragma unroll
                            for (int u = 0; u < CS; ++u)
#pragma unroll
                                for (int r = 0; r < R; ++r)
#pragma unroll
                                    for (int v = 0; v < 4; ++v) {
                                        const float x = gm[u][r][v];
                                        if (x != 0.0f && __builtin_isfinite(x))
                                            atomicAdd(&B64k[(size_t)oc[u] * NP + quad_t(16 * r + 4 * g + v)], to_fixed(x, F));
                                    }
                        }
                        if (c.t0 < CS) {  // the sequences' first steps
#pragma unroll
                            for (int r = 0; r < R; ++r)
#pragma unroll
                                for (int v = 0; v < 4; ++v) {
                                    const int i = 16 * r + 4 * g + v;
                                    float x = 0.0f;
#pragma unroll
                                    for (int u = 0; u < CS; ++u) x = c.t0 == u ? gm[u][r][v] : x;
                                    if (i < N) add_fixed_slots(&a.pi64[(size_t)k * N + i], x, F, &a.nanflag[k], sl);
                                }
                        }
                    };
                    Chunk cp{0, 0};
                    int half_ring = 0;
                    for (int p = 0; p <= nseg; ++p) {
                        const int j = nseg - p;
                        const float4 *sa = seg_alpha(j);
                        segment_barrier();
                        for (int s = 0; s < nch; ++s, half_ring ^= 1) {
                            const Chunk cn = back_chunk(j, s);
#pragma unroll
                            for (int u = 0; u < CS; ++u) {
#pragma unroll
                                for (int r = 0; r < R; ++r)
                                    an[u][r] = sa[(size_t)(max(cn.n - 1 - u, 0) * R + r) * WAVE + lane];
                                on[u] = load_sym(cn.t0 - u);
                            }
                            if (cp.n > 0) take(cp, half_ring ^ 1);
#pragma unroll
                            for (int u = 0; u < CS; ++u) {
                                oc[u] = checked(on[u]);
#pragma unroll
                                for (int r = 0; r < R; ++r) ac[u][r] = an[u][r];
                            }
                            cp = cn;
                            lds_barrier();
                        }
                    }
                    if (cp.n > 0) take(cp, half_ring ^ 1);
                    if (!__builtin_isfinite(nan_acc)) atomicOr(&a.nanflag[k], 1);
                }
            }  // Tmax > 0
            if (NBLDS) {
                // the tile's emission partial into its slab slot (zeros for an empty tile)
                __syncthreads();
                const int64_t slot = slab_slot(gbeg, k, tile);
                float *dst = a.slab + (size_t)(dbg_in(slot, slab_slots(a.S, a.K), HMM_DEBUG_SLAB) ? slot : 0) * M * NP;
                for (int idx = threadIdx.x; idx < M * NP; idx += ROLES * WAVE) {
                    const int o = idx / NP, ic = idx % NP;
                    dst[(size_t)o * NP + (ic ^ (o * 4 & swz))] = nbl[idx];
                    nbl[idx] = 0.0f;
                }
            }
        }
    }
}

constexpr size_t LDS_CU = 160 * 1024;

// LDS for the emission partial of a workgroup: the [M][NP] sums, then the slot masks.
size_t partial_bytes(int NP, int M) { return (size_t)M * NP * 4 + (size_t)((M + 1) / 2) * 4; }

// Which variant a shape takes: the emission partial in LDS (when it fits and the slab of
// per-tile partials stays within SLAB_MAX_BYTES), else adds to the global counts.  Beside the
// rings it fits up to 2317 symbols at 16 states, 1105 at 32 and 692 at 48.  Counts of 4 models, 300
// sequences of 50-800 and 8000 of 20-300, last shape in LDS and first in memory: 16 states 468
// and 643 us, 254 and 399; 32 states 792 and 1030, 415 and 793; 48 states 1336 and 1518, 669 and
// 1135.
template <int R>
bool use_partial(int M, int S, int K) {
    if (slab_slots(S, K) * M * 16 * R * 4 > SLAB_MAX_BYTES) return false;
    return partial_bytes(16 * R, M) + AdjShape<R, 2>::static_bytes <= LDS_CU;
}

// Workgroups per CU that the tiles can fill, within what the registers allow.
template <int R>
int want_per_cu(int S, int K, int cu_count) {
    const int64_t n = (tile_bound(S, K, false, TILE) + cu_count - 1) / cu_count;
    return (int)std::min<int64_t>(std::max<int64_t>(n, 1), adj_waves(R, 2));
}

// The kernel and LDS of a launch, and the grid that the card holds at once.
struct AdjPlan {
    void (*kern)(DevPtrs, AdjLaunch);
    size_t lds;
    int grid;
};

template <int R>
AdjPlan plan_for(int M, int S, int cu_count, int K) {
    AdjPlan p{k_adj_tile<R, false, 2>, 0, 0};
    if (use_partial<R>(M, S, K)) {
        const int want = want_per_cu<R>(S, K, cu_count);
        // Four steps per chunk halve the barriers of a tile that has its CU to itself: with four
        // and two, 174 and 184 us for an EM iteration on 147 sequences of 20-200 (6 models, 5 states),
        // 890 and 924 on 300 of 20-1500 (8 states, 30 symbols), 273 and 272 on 2000 of 50-400 (12
        // models, 16 states).  With more of them on a CU two steps take fewer registers and less LDS:
        // 1361 and 962 us (40000 sequences of 50-600, 8 states, 6 symbols), 1005 and 733 (16
        // states, 64 symbols), 295 and 284 (4096 of 50-400).
        constexpr int WIDE = R == 1 ? 4 : 2;
        if (want == 1 && partial_bytes(16 * R, M) + AdjShape<R, WIDE>::static_bytes <= LDS_CU) {
            p.kern = k_adj_tile<R, true, WIDE>;
        } else {
            p.kern = k_adj_tile<R, true, 2>;
        }
        p.lds = partial_bytes(16 * R, M);
        if (p.lds > 64 * 1024)
            (void)hipFuncSetAttribute((const void *)p.kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)p.lds);
    }
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, p.kern, ROLES * WAVE, p.lds) != hipSuccess || per_cu < 1)
        per_cu = 1;
    p.grid = cu_count * per_cu;
    if (K > 0 && p.grid >= K) p.grid = (p.grid / K) * K;
    return p;
}

template <int R>
hipError_t launch_r(const DevPtrs &d, const AdjLaunch &a, int cu_count, hipStream_t st) {
    const AdjPlan p = plan_for<R>(a.M, a.S, cu_count, a.K);
    const int grid = persistent_grid(p.grid, tile_bound(a.S, a.K, false, TILE), 1, a.K, a.max_grid);
    if (grid > a.seg_slots) return hipErrorInvalidValue;
    if (use_partial<R>(a.M, a.S, a.K) ? a.slab == nullptr : a.B64 == nullptr) return hipErrorInvalidValue;
    p.kern<<<grid, ROLES * WAVE, p.lds, st>>>(d, a);
    return hipGetLastError();
}

}  // namespace

bool adj_mfma_supported(int NP) { return NP == 16 || NP == 32 || NP == 48; }

bool adj_mfma_slab(int NP, int M, int S, int K) {
    switch (NP / 16) {
        case 1: return use_partial<1>(M, S, K);
        case 2: return use_partial<2>(M, S, K);
        case 3: return use_partial<3>(M, S, K);
        default: return false;
    }
}

int adj_mfma_slots(int NP, int M, int S, int K, int cu_count) {
    switch (NP / 16) {
        case 1: return plan_for<1>(M, S, cu_count, K).grid;
        case 2: return plan_for<2>(M, S, cu_count, K).grid;
        case 3: return plan_for<3>(M, S, cu_count, K).grid;
        default: return 0;
    }
}

int64_t adj_mfma_seg_stride(int NP, int max_len) {
    int L = 1;
    while ((int64_t)L * L < max_len) ++L;
    return (int64_t)2 * L * WAVE * (4 * (NP / 16) + 1);
}

hipError_t launch_adj_mfma(const DevPtrs &d, const AdjLaunch &a, int cu_count, hipStream_t st) {
    switch (a.NP / 16) {
        case 1: return launch_r<1>(d, a, cu_count, st);
        case 2: return launch_r<2>(d, a, cu_count, st);
        case 3: return launch_r<3>(d, a, cu_count, st);
        default: return hipErrorInvalidValue;
    }
}

HMM_DEBUG_TAKE(debug_take_adj_mfma)

}  // namespace hmm
