// Data partition by products on the matrix cores (a variant beyond the paper's listing,
// see k_onehot in gt_kernels.hpp for the protocol):
//   sel[k][i] = sum_r L[r][i] * OH[r][k]     (op, zero sharing of stream 0, word k*N8+i, reshare)
//   M[i]     <- 2 M[i] + sum_k sel[k][i] * X[k][i] + 1   (op+1, zero sharing of stream 0, word i, reshare)
// fused in one launch: a workgroup = the three parties' wavefronts works on a block of 32
// samples; each wavefront computes its party's three-term product
//   L_p (OH_p + OH_{p+1}) + L_{p+1} OH_p
// as an int8-limb GEMM (64 columns x 32 samples per pass, contraction over the nodes r of
// both terms), adds the zero sharing, sends its component to the predecessor through LDS
// and accumulates the row inner product with X; sel never reaches device memory.
//
// Operands.  OH comes as limb bytes with the node index contiguous (k_onehot or k_oh_limbs): that is the
// A operand as it is.  L lives in the limb tiles of the statistics contraction, where the
// SAMPLES are contiguous ([block][limb][row r][32 samples]); the matrix core wants the
// contraction index contiguous per lane, so every 32 x 32 byte tile is transposed through a
// small wavefront-private LDS area: dword columns are written with a padded stride, lanes
// read 16 dwords of their sample's dword column and pick their byte with byte permutes.
#pragma once
#include "gt_kernels.hpp"

// OH as limb bytes, see k_onehot
__global__ __launch_bounds__(256) void k_oh_limbs(P6 OH, unsigned char *OHL, u32 np, u32 d, u32 rpad, u32 dpad)
{
    const u64 per = (u64)dpad * rpad, total = 6 * per;
    for (u64 t = (u64)blockIdx.x * blockDim.x + threadIdx.x; t < total; t += (u64)gridDim.x * blockDim.x) {
        const u32 pw = (u32)(t / per), k = (u32)((t % per) / rpad), r = (u32)(t % rpad), p = pw >> 1, w = pw & 1;
        u64 x = 0;
        if (r < np && k < d) x = OH.o[p][(u64)r * d + k] + (w ? 0 : OH.n[p][(u64)r * d + k]);
        const u64 y = (x + GT_BIAS) ^ GT_BIAS;
#pragma unroll
        for (int s = 0; s < 8; s++) OHL[(((u64)pw * 8 + s) * dpad + k) * rpad + r] = (unsigned char)(y >> (8 * s));
    }
}

#define PM_TP_STRIDE 36                      // dwords between the dword columns of the transpose area
#define PM_TP_WORDS (8 * PM_TP_STRIDE)       // dwords per area

struct PartMmArgs {
    KCommon c;                 // c.op: the column-selection op; c.op + 1: the row inner product
    LimbTri L;                 // leaf one-hot of the previous level, one matrix per component
    const unsigned char *OHL;
    P6 XT, M;
    u64 N, N8, nblk;
    u32 d, dpad, rpad;         // columns, padded to 64; node rows padded to 32
};

// Zero-sharing words under the party's own key for one pass of the epilogue: pass covers the 16 rows
// m = pass*16 + ri, ri < 16, of the 64 x 32 tile; lane l evaluates the block of row ri = l/4, sample
// group l%4; words to scr[m*32 + sample].  The words under the next key are the next party's, in its
// scratch (evaluating both keys per party took twice the passes: 154 us a level
// for 19,997 x 101, 131 us now).
__device__ __forceinline__ void pm_prf_pass(const PartMmArgs &a, const Key &own, u64 *scr, u32 pass, u32 kg, u64 ib, u32 lane)
{
    const u32 m = pass * 16 + (lane >> 2), g = lane & 3;
    const u64 kcol = (u64)kg * 64 + m;
    u64 blk[8];
    chacha8(own, ((kcol * a.N8 + ib * 32) >> 3) + g, a.c.op, 0, blk);
#pragma unroll
    for (int q = 0; q < 8; q++) scr[m * 32 + g * 8 + q] = blk[q];
}

// More than GT_PM16_NODES nodes in the level before.  Bound: vector work (the PRF, recombination, byte permutes) beside matrix-core time, one wavefront per SIMD on three of a
// compute unit's four: 256 accumulators leave room for no second workgroup, and 45 registers spill (184 B a lane).
__global__ __launch_bounds__(192, 1) void k_part_mm(PartMmArgs a)
{
    __shared__ u64 s_wire[GT_LWIRE_WORDS];
    __shared__ u64 s_cnt[6];
    __shared__ u64 s_prf[3][64 * 32];            // per party: the zero-sharing words of a 64 x 32 tile under its own key
    __shared__ u64 s_x[3][16 * GT_LANES];        // the reshared components, 16 per lane and exchange
    __shared__ u32 s_tp[3][2 * PM_TP_WORDS];     // two transpose areas per wavefront, used alternately
    const int p = party_of_wave(), lane = threadIdx.x, pn = p == 2 ? 0 : p + 1;
    LWire W; W.init(s_wire, s_cnt);
    const Key own = load_key(a.c.keys, p);
    u64 *scr = s_prf[p];
    const u64 *scrn = s_prf[pn];
    u32 *tp = s_tp[p];
    const u32 n = lane & 31, hi = (u32)lane >> 5;
    const Sh one = pub(p, 1);
    const u32 bsel = (n & 3) | ((4 + (n & 3)) << 8) | 0x0c0c0000u;   // byte n%4 of two dwords into bytes 0 and 1
    const u32 nrc = a.rpad / 32, nkg = a.dpad / 64, nch = 2 * nrc;
    for (u64 ib = blockIdx.x; ib < a.nblk; ib += gridDim.x) {
        const u64 i = ib * 32 + n;
        const bool ilive = i < a.N;
        u64 dacc = 0;
        for (u32 kg = 0; kg < nkg; kg++) {
            v16i acc[8][2];
#pragma unroll
            for (int u = 0; u < 8; u++)
#pragma unroll
                for (int t = 0; t < 2; t++)
#pragma unroll
                    for (int v = 0; v < 16; v++) acc[u][t][v] = 0;
            // chunks of 32 node rows: first those of L_p x (OH own+next), then those of L_{p+1} x OH own.
            // The eight limb tiles of the next chunk are in flight while this one is transposed and
            // multiplied (the last iteration loads its own chunk again, unused, so that the number of
            // loads in flight at every wait is the same).  The four passes of the epilogue's zero-sharing
            // words go one with each chunk, in the shadow of its matrix-core instructions; with the two
            // chunks of at most 32 nodes two passes are left for after the loop, from the fifth chunk on
            // words already there are evaluated again, because a branch or a second loop takes the passes out
            // of the schedule of the first four chunks (19,997 x 101 with up to 32, 64, 256 nodes in the
            // level before: 131, 155, 346 us like this; with a branch 165, 211, 520; with a second loop 205,
            // 228, 410).
            v4i xn[8];
#define PM_LOAD(X, CH)                                                                               \
            {                                                                                        \
                const u32 w_ = (CH) / nrc, rc_ = (CH) % nrc;                                         \
                const u32 j_ = (u32)p + w_ >= 3 ? 0 : (u32)p + w_;                                   \
                const LimbMat LM_ = j_ == 0 ? a.L.m[0] : (j_ == 1 ? a.L.m[1] : a.L.m[2]);            \
                _Pragma("unroll") for (int s = 0; s < 8; s++)                                        \
                    X[s] = *(const v4i *)(LM_.base + limb_addr(LM_, ib, s, (u64)rc_ * 32) + (lane >> 1) * 32 + (lane & 1) * 16); \
            }
            PM_LOAD(xn, 0)
            for (u32 ch = 0; ch < nch; ch++) {
                const u32 w = ch / nrc, rc = ch % nrc;
                v4i x[8], A[2][8];
#pragma unroll
                for (int s = 0; s < 8; s++) x[s] = xn[s];
                PM_LOAD(xn, (ch + 1 < nch ? ch + 1 : ch))
#pragma unroll
                for (int t = 0; t < 2; t++) {
                    const u64 col = (u64)kg * 64 + t * 32 + n;
#pragma unroll
                    for (int s = 0; s < 8; s++)
                        A[t][s] = *(const v4i *)(a.OHL + ((((u64)(p * 2 + w) * 8 + s) * a.dpad + col) * a.rpad + rc * 32 + hi * 16));
                }
                // B operand: the eight limb tiles [32 rows r][32 samples] of this chunk, transposed
                v4i Bt[8];
#pragma unroll
                for (int s = 0; s < 8; s++) {
                    __builtin_amdgcn_wave_barrier();
#pragma unroll
                    for (int q = 0; q < 4; q++) tp[(s & 1) * PM_TP_WORDS + ((lane & 1) * 4 + q) * PM_TP_STRIDE + (lane >> 1)] = (u32)x[s][q];
                    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                    __builtin_amdgcn_wave_barrier();
                    u32 dw[16];
#pragma unroll
                    for (int jj = 0; jj < 4; jj++) {
                        const v4i y = *(const v4i *)&tp[(s & 1) * PM_TP_WORDS + (n >> 2) * PM_TP_STRIDE + hi * 16 + jj * 4];
                        dw[jj * 4 + 0] = (u32)y[0]; dw[jj * 4 + 1] = (u32)y[1]; dw[jj * 4 + 2] = (u32)y[2]; dw[jj * 4 + 3] = (u32)y[3];
                    }
                    v4i o;
#pragma unroll
                    for (int q = 0; q < 4; q++) {
                        const u32 lo2 = __builtin_amdgcn_perm(dw[4 * q + 1], dw[4 * q + 0], bsel);
                        const u32 hi2 = __builtin_amdgcn_perm(dw[4 * q + 3], dw[4 * q + 2], bsel);
                        o[q] = (int)__builtin_amdgcn_perm(hi2, lo2, 0x05040100u);
                    }
                    Bt[s] = o;
                }
                pm_prf_pass(a, own, scr, ch & 3, kg, ib, (u32)lane);
#pragma unroll
                for (int t = 0; t < 2; t++)
#pragma unroll
                    for (int s = 0; s < 8; s++)
#pragma unroll
                        for (int u = 0; u < 8 - s; u++)
                            acc[s + u][t] = __builtin_amdgcn_mfma_i32_32x32x32_i8(A[t][s], Bt[u], acc[s + u][t], 0, 0, 0);
                // one matrix-core instruction, then half a dozen vector instructions of the PRF, and so on
#pragma unroll
                for (int q = 0; q < 72; q++) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x002, 6, 0);
                }
            }
#undef PM_LOAD
            // the samples' own values for the epilogue, on their way while the remaining words are evaluated
            Sh xv[2][16];
            u32 nl = 0;
#pragma unroll
            for (int t = 0; t < 2; t++)
#pragma unroll
                for (int v = 0; v < 16; v++) {
                    const u64 kcol = (u64)kg * 64 + t * 32 + 8 * (v >> 2) + hi * 4 + (v & 3);
                    const bool live = ilive && kcol < a.d;
                    nl += live ? 1u : 0u;
                    xv[t][v] = live ? ld(a.XT, p, kcol * a.N8 + i) : Sh{ 0, 0 };
                }
            for (u32 pass = nch; pass < 4; pass++) pm_prf_pass(a, own, scr, pass, kg, ib, (u32)lane);   // fewer than four chunks
            W.nresh += 64u * nl;
            __syncthreads();                             // every party's words are there
            // epilogue, one half of the tile (32 columns, 16 per lane) at a time: recombine the limb
            // levels, add the zero sharing, send the component to the predecessor, inner product with X
#pragma unroll
            for (int t = 0; t < 2; t++) {
                u64 snd[16];
#pragma unroll
                for (int v = 0; v < 16; v++) {
                    u64 z = 0;
#pragma unroll
                    for (int u = 0; u < 8; u++) z += (u64)(long long)acc[u][t][v] << (8 * u);
                    const u32 m = t * 32 + 8 * (v >> 2) + hi * 4 + (v & 3);
                    snd[v] = z + (scr[m * 32 + n] - scrn[m * 32 + n]);
                    s_x[p][v * GT_LANES + lane] = snd[v];
                }
                __syncthreads();
#pragma unroll
                for (int v = 0; v < 16; v++) {
                    const Sh sel = { snd[v], s_x[pn][v * GT_LANES + lane] };
                    dacc += prod3(sel, xv[t][v]);                       // X is zero where the element does not exist
                }
                __syncthreads();
            }
        }
        // the two halves of the wavefront hold the sums over different rows of the same sample
        dacc += (u64)__shfl_xor((unsigned long long)dacc, 32, GT_LANES);
        {
            // zero sharing of the inner product: words ib*32 .. +31 of stream 0 under op+1, four blocks
            if (lane < 4) {
                u64 blk[8];
                chacha8(own, ib * 4 + lane, a.c.op + 1, 0, blk);
#pragma unroll
                for (int q = 0; q < 8; q++) scr[lane * 8 + q] = blk[q];
            }
            __syncthreads();
        }
        Sh z;
        z.o = dacc + (scr[n] - scrn[n]);
        z.n = W.reshare1(z.o, (ilive && hi == 0) ? 64u : 0u);
        if (ilive && hi == 0) st(a.M, p, i, scale(ld(a.M, p, i), 2) + z + one);
        __syncthreads();                         // the message slots and the scratch are rewritten by the next block
        W.drain();
    }
    W.flush(a.c.wire);
}

// ---------------------------------------------------------------------------------
// The same for at most GT_PM16_NODES nodes in the level before: both terms' nodes, 2 x 32, are the contraction of one
// v_mfma_i32_16x16x64_i8, so a party's wavefront keeps the limbs of its 16 samples in 32 registers for all columns and a
// tile of 16 columns needs 32 accumulators instead of the 256 that leave a SIMD of k_part_mm to one wavefront.  A step covers
// 32 columns x 16 samples: one PRF pass, 72 matrix-core instructions, two barriers.
// Bound: the vector ALU (PRF, recombination, three-term products) and the reads of X, with three wavefronts per SIMD.
// 19,997 samples x 101 columns, 1 to 32 nodes in the level before: 131 us a level with k_part_mm, 51 now (with two wavefronts
// per SIMD 56, with four, which spill 100 registers, 90; with three 3 spill).
#define GT_PM16_NODES 32
#define PM16_STRIDE 80                       // bytes between the samples of a limb in the staging area (64 and a pad)
__global__ __launch_bounds__(192, 3) void k_part_mm16(PartMmArgs a)
{
    union Stage { unsigned char limb[8 * 16 * PM16_STRIDE]; struct { u64 prf[8 * GT_LANES], x[8 * GT_LANES]; }; };
    __shared__ Stage s_w[3];                     // first the samples' limbs, then zero-sharing words under the party's own key and messages
    __shared__ u64 s_cnt[6];
    const int p = party_of_wave(), pn = p == 2 ? 0 : p + 1;
    const u32 lane = threadIdx.x, n = lane & 15, kq = lane >> 4;
    LWire W; W.init(nullptr, s_cnt);
    const Key own = load_key(a.c.keys, p);
    const u64 i0 = (u64)blockIdx.x * 16, i = i0 + n;
    const bool ilive = i < a.N;
    const u64 *xpo = own_of(a.XT, p), *xpn = nxt_of(a.XT, p), ic = ilive ? i : a.N - 1;
    // L: lane = (term, node), 16 samples of a limb per load; afterwards lane = (sample, 16 of the 64 nodes of both terms)
    v4i B[8];
    {
        const int j = lane < 32 ? p : pn;
        const LimbMat m = j == 0 ? a.L.m[0] : (j == 1 ? a.L.m[1] : a.L.m[2]);
        v4i x[8];
#pragma unroll
        for (int s = 0; s < 8; s++) x[s] = *(const v4i *)(m.base + limb_addr(m, i0 >> 5, s, lane & 31) + (i0 & 31));
        unsigned char *st = s_w[p].limb + lane;
#pragma unroll
        for (int s = 0; s < 8; s++)
#pragma unroll
            for (int q = 0; q < 16; q++) st[(s * 16 + q) * PM16_STRIDE] = (unsigned char)((u32)x[s][q >> 2] >> (8 * (q & 3)));
        wave_sync();
#pragma unroll
        for (int s = 0; s < 8; s++) B[s] = *(const v4i *)(s_w[p].limb + (s * 16 + n) * PM16_STRIDE + kq * 16);
        wave_sync();
    }
    // the columns' limbs: row = column, own + next part with the first term's nodes, own part with the second's
    const unsigned char *A0 = a.OHL + ((u64)(p * 2 + (kq >> 1)) * 8 * a.dpad + n) * a.rpad + (kq & 1) * 16;
    u64 dacc = 0;
    for (u32 k0 = 0; k0 < a.d; k0 += 32) {
        {
            u64 blk[8];
            chacha8<PRF_PAIR>(own, (((u64)(k0 + (lane >> 1)) * a.N8 + i0) >> 3) + (lane & 1), a.c.op, 0, blk);
#pragma unroll
            for (int s = 0; s < 8; s++) s_w[p].prf[lane * 8 + s] = blk[s];
        }
        u64 z[8];
        Sh x[8];
#pragma unroll
        for (int t = 0; t < 2; t++) {
            v4i A[8], acc[8];
#pragma unroll
            for (int s = 0; s < 8; s++) A[s] = *(const v4i *)(A0 + ((u64)s * a.dpad + k0 + t * 16) * a.rpad);
#pragma unroll
            for (int v = 0; v < 4; v++) {
                // (an existing element where this one does not exist: a load without a branch, cleared below)
                const u32 k = k0 + t * 16 + kq * 4 + v;
                const u64 e = (u64)(k < a.d ? k : a.d - 1) * a.N8 + ic;
                x[t * 4 + v].o = xpo[e]; x[t * 4 + v].n = xpn[e];
            }
#pragma unroll
            for (int u = 0; u < 8; u++) acc[u] = v4i{ 0, 0, 0, 0 };
#pragma unroll
            for (int s = 0; s < 8; s++)
#pragma unroll
                for (int u = 0; u < 8 - s; u++) acc[s + u] = __builtin_amdgcn_mfma_i32_16x16x64_i8(A[s], B[u], acc[s + u], 0, 0, 0);
#pragma unroll
            for (int v = 0; v < 4; v++) {
                u64 r = 0;
#pragma unroll
                for (int u = 0; u < 8; u++) r += (u64)(long long)acc[u][v] << (8 * u);
                z[t * 4 + v] = r;
            }
        }
        __syncthreads();                             // every party's words are there
#pragma unroll
        for (int v = 0; v < 8; v++) {
            const u32 w = ((v >> 2) * 16 + kq * 4 + (v & 3)) * 16 + n;
            z[v] += s_w[p].prf[w] - s_w[pn].prf[w];
            s_w[p].x[v * GT_LANES + lane] = z[v];
        }
#pragma unroll
        for (int v = 0; v < 8; v++) {
            const bool live = ilive && k0 + (v >> 2) * 16 + kq * 4 + (v & 3) < a.d;
            W.nresh += live ? 64u : 0u;
            x[v].o = live ? x[v].o : 0; x[v].n = live ? x[v].n : 0;
        }
        __syncthreads();
#pragma unroll
        for (int v = 0; v < 8; v++) dacc += prod3(Sh{ z[v], s_w[pn].x[v * GT_LANES + lane] }, x[v]);
    }
    // the lanes of a sample hold the sums over different columns
    dacc += (u64)__shfl_xor((unsigned long long)dacc, 16, GT_LANES);
    dacc += (u64)__shfl_xor((unsigned long long)dacc, 32, GT_LANES);
    __syncthreads();                                 // the last messages have been read
    if (lane < 2) {                                  // zero sharing of the inner product: words i0 .. i0 + 15 of stream 0 under op + 1
        u64 blk[8];
        chacha8(own, (i0 >> 3) + lane, a.c.op + 1, 0, blk);
#pragma unroll
        for (int q = 0; q < 8; q++) s_w[p].prf[lane * 8 + q] = blk[q];
    }
    __syncthreads();
    Sh z = { dacc + (s_w[p].prf[n] - s_w[pn].prf[n]), 0 };
    s_w[p].x[lane] = z.o;
    W.nresh += ilive && kq == 0 ? 64u : 0u;
    __syncthreads();
    z.n = s_w[pn].x[lane];
    if (ilive && kq == 0) st(a.M, p, i, scale(ld(a.M, p, i), 2) + z + pub(p, 1));
    W.flush(a.c.wire);
}
