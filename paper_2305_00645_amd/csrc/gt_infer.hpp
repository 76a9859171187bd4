// Oblivious inference in one launch (Sec. V-C of the GTree paper).  The H iterations of an
// instance - array access over the level's slice of the tree, array access into the
// instance's own features, optional threshold comparison, index update - and the final
// access over the leaf labels do not interact with any other instance, so a workgroup
// carries a tile of instances through all of them: no per-level launches, no partial sums
// in device memory, no workspace.  Operation ids, element indices (k*N8 + i) and streams are
// those of the level-by-level path, so every share is the same.
#pragma once
#include "gt_kernels.hpp"

struct InferArgs {
    KCommon c;                 // c.op: first operation id of the batch
    P6 feat, thr, leaf;        // per tree 2^H-1 ids, 2^H-1 thresholds (THR), 2^H labels, tree after tree
    P6 I, out;                 // NI x d row-major instances; results out[t*NI + i]
    u64 NI, N8;
    u32 d, H, ntrees;          // ntrees > 1: a forest; tree t takes the operation ids that the t-th of
                               // ntrees single-tree batches in a row would take
    u32 noct;                  // groups of 8 instances per tile, at most GT_INFER_OCT(NW)
};

// A workgroup is NW wavefronts (1, 2 or 4), each with the three parties in 21 lanes (WWire).  Its 21 NW lanes per party split into noct groups of 8
// instances x ncol columns: lane (o, cl) tests the 8 instances of group o against columns cl, cl + ncol, ... of the current access and adds up its
// share of the inner products in registers; the ncol partial sums meet in LDS.  The messages of
// the tests stay inside a wavefront; the workgroup synchronises three times per access, where the
// offline and zero-sharing words of the rows, evaluated by all lanes side by side, and the sums
// change hands.
#define GT_INFER_LANES(NW) ((NW) * GT_TP)
#define GT_INFER_OCT(NW) (4 * (NW))          // groups of a workgroup at most: 19 KB of LDS per wavefront, two per SIMD
// words per group of 8 instances.  Material of an access: r's arithmetic and Boolean components
// [6][8], zero-sharing words [2 streams][3 keys][8]; of a comparison: [9][8] components (r, r's bits,
// beta), beta's bits [8], mask words [2][3][8].  Values: index, id, threshold as [party][own, next][8].
#define GT_INFER_MAT 128
#define GT_INFER_VAL 48

template <int ISSUE>
struct InferWg {
    EqWave E;
    u64 *mat, *val, *sum;        // of this lane's group: GT_INFER_MAT, 3 * GT_INFER_VAL, [2][3][8] words
    const u32 *keys;
    u32 cl, ncol;
    u64 ngrp, grp, NI;           // groups of the batch, this lane's group
    bool active, one;            // the lane has a group / is the one that counts and stores for its group and party
    int p, pn;

    __device__ __forceinline__ u64 &value(int which, int party, int comp, int s) { return val[which * GT_INFER_VAL + (party * 2 + comp) * 8 + s]; }
    __device__ __forceinline__ u32 live() const { return grp < ngrp ? live8(grp * 8, NI) : 0u; }

    // the PRF block of role b: block `blk` of a stream under a key; which lanes evaluate it is free
    __device__ __forceinline__ void block(int key, u64 blk, u32 op, u32 stream, u64 (&D)[8])
    {
        Key kv;
#pragma unroll
        for (int i = 0; i < 8; i++) kv.k[i] = keys[key * 8 + i];
        chacha8<ISSUE>(kv, blk, op, stream, D);
    }

    // One array access: E[k] = [u - base == k] for k < w, converted to arithmetic, and
    // z = sum_k E[k] * W1[off + k] (ROWS: * the instance's own feature k), z2 likewise with W2
    // (NDOT = 2, where nd2 is set); zero sharing of stream 2 (3), word i; one reshare round.
    // u: value `which`.
    template <bool ROWS, int NDOT>
    __device__ __forceinline__ void access(u32 op, int which, u64 base, u32 w, const P6 &W1, const P6 &W2, u64 off, bool nd2,
                                           const P6 &I, u32 d, u64 (&zo)[8], u64 (&zn)[8], u64 (&z2o)[8], u64 (&z2n)[8])
    {
        WWire &W = E.W;
        const Sh pub1 = pub(p, 1);
        const u32 k1o = (u32)pub1.o + 1, k1n = (u32)pub1.n + 1, nroles = 8 + 3 * (nd2 ? 2 : 1);
        __syncthreads();                               // the previous access has read its material
        for (u32 b0 = 0; b0 < nroles; b0 += 3 * ncol) {
            const u32 b = b0 + cl * 3 + (u32)p;
            if (active && b < nroles) {
                u64 D[8];
                const u32 q = b < 8 ? 0 : (b - 8) / 3;
                const int key = b < 8 ? GT_KEY_DEALER : (int)(b - 8 - 3 * q);
                block(key, b < 8 ? grp * 8 + b : grp, op, b < 8 ? 0 : 2 + q, D);
                if (b < 8) {
                    mat[b] = D[1]; mat[8 + b] = D[2]; mat[16 + b] = D[0] - D[1] - D[2];
                    mat[24 + b] = D[3]; mat[32 + b] = D[4]; mat[40 + b] = D[0] ^ D[3] ^ D[4];
                } else {
#pragma unroll
                    for (int s = 0; s < 8; s++) mat[48 + (b - 8) * 8 + s] = D[s];
                }
            }
        }
        if (active && cl == 0) {
#pragma unroll
            for (int s = 0; s < 8; s++) { sum[p * 8 + s] = 0; if (NDOT == 2) sum[24 + p * 8 + s] = 0; }
        }
        __syncthreads();
        // the one opening of the access: c = u + r - base is public afterwards; the lanes of a group
        // replay the same message, one of them counts
        u64 cpub[8], rho_o[8], rho_n[8];
        {
            u64 snd[8], mn[8], rcv[8];
#pragma unroll
            for (int s = 0; s < 8; s++) {
                snd[s] = value(which, p, 0, s) + mat[p * 8 + s]; mn[s] = value(which, p, 1, s) + mat[W.pn * 8 + s];
                rho_o[s] = mat[24 + p * 8 + s]; rho_n[s] = mat[24 + W.pn * 8 + s];
            }
            W.open64<8>(snd, rcv);
            W.nopen += one ? 64u * live() : 0u;
#pragma unroll
            for (int s = 0; s < 8; s++) cpub[s] = snd[s] + mn[s] + rcv[s] - base;
        }
        u64 acc[8], acc2[8], xo[8], xn[8];
#pragma unroll
        for (int s = 0; s < 8; s++) { acc[s] = 0; acc2[s] = 0; }
        const u64 *xpo = nullptr, *xpn = nullptr;
        u64 last = 0;                                  // rows beyond the batch read its last one
        if (ROWS) { xpo = own_of(I, p); xpn = nxt_of(I, p); last = NI - 1; }
        const auto fetch_x = [&](u32 k) {
            const u32 col = k < d ? k : d - 1;
#pragma unroll
            for (int s = 0; s < 8; s++) {
                const u64 i = grp * 8 + s < last ? grp * 8 + s : last;
                xo[s] = xpo[i * d + col]; xn[s] = xpn[i * d + col];
            }
        };
        const u64 *w1o = nullptr, *w1n = nullptr, *w2o = nullptr, *w2n = nullptr;
        if (!ROWS) { w1o = own_of(W1, p) + off; w1n = nxt_of(W1, p) + off; }
        if (!ROWS && NDOT == 2) { w2o = own_of(W2, p) + (nd2 ? off : 0); w2n = nxt_of(W2, p) + (nd2 ? off : 0); }
        if (ROWS) fetch_x(cl);
        for (u32 k0 = 0; k0 < w; k0 += ncol) {
            const u32 col = k0 + cl;
            const bool act = active && col < w;
            Sh Wk = { 0, 0 }, Wk2 = { 0, 0 };
            u64 cd[8];
#pragma unroll
            for (int s = 0; s < 8; s++) cd[s] = cpub[s] - col;
            const u32 f = E.template tests<false, ISSUE>(op, (u64)col * ngrp + grp, cd, rho_o, rho_n, 0, 0, act ? live() : 0u, [&]() {
                if (!ROWS && act) { Wk.o = w1o[col]; Wk.n = w1n[col]; }
                if (!ROWS && NDOT == 2 && act && nd2) { Wk2.o = w2o[col]; Wk2.n = w2n[col]; }
            });
            if (ROWS) {
#pragma unroll
                for (int s = 0; s < 8; s++) {
                    const u32 m = (u32)((int)(f << (31 - eq_pos(s))) >> 31);
                    const Sh e = { eq_select(E.row(p, s), m, k1o), eq_select(E.row(W.pn, s), m, k1n) }, x = { xo[s], xn[s] };
                    if (act) acc[s] += prod3(e, x);
                }
                fetch_x(k0 + ncol + cl);
            } else {
                // columns beyond w: W = 0, the sum stays (see k_eqgrid)
                const u64 S = Wk.o + Wk.n, nc = ~(pub1.o * S + pub1.n * Wk.o);
                const u64 S2 = Wk2.o + Wk2.n, nc2 = ~(pub1.o * S2 + pub1.n * Wk2.o);
#pragma unroll
                for (int s = 0; s < 8; s++) {
                    const u32 m = (u32)((int)(f << (31 - eq_pos(s))) >> 31);
                    const u64 mm = (u64)m | ((u64)m << 32), bo = E.row(p, s), bn = E.row(W.pn, s);
                    acc[s] += ((mm & nc) + bo * S + bn * Wk.o) ^ mm;
                    if (NDOT == 2) acc2[s] += ((mm & nc2) + bo * S2 + bn * Wk2.o) ^ mm;
                }
            }
        }
        if (active && W.real) {
#pragma unroll
            for (int s = 0; s < 8; s++) {
                atomicAdd((unsigned long long *)&sum[p * 8 + s], (unsigned long long)acc[s]);
                if (NDOT == 2 && nd2) atomicAdd((unsigned long long *)&sum[24 + p * 8 + s], (unsigned long long)acc2[s]);
            }
        }
        __syncthreads();
        // every lane of a group finishes the group's result
#pragma unroll
        for (int s = 0; s < 8; s++) zo[s] = sum[p * 8 + s] + (mat[48 + p * 8 + s] - mat[48 + W.pn * 8 + s]);
        W.reshare64<8>(zo, zn);
        W.nresh += one ? 64u * live() : 0u;
        if (NDOT == 2 && nd2) {
#pragma unroll
            for (int s = 0; s < 8; s++) z2o[s] = sum[24 + p * 8 + s] + (mat[72 + p * 8 + s] - mat[72 + W.pn * 8 + s]);
            W.reshare64<8>(z2o, z2n);
            W.nresh += one ? 64u * live() : 0u;
        }
    }

    // index <- 2 index + [x > theta] + 1 (threshold mode): x and theta are values 1 and 2; the lanes of
    // a group share out its 8 instances
    __device__ __forceinline__ void greater(u32 op)
    {
        WWire &W = E.W;
        __syncthreads();                               // x, theta stored; the access's material has been read
        for (u32 b0 = 0; b0 < 14; b0 += 3 * ncol) {
            const u32 b = b0 + cl * 3 + (u32)p;
            if (active && b < 14) {
                u64 D[8];
                const u32 q = b < 8 ? 0 : (b - 8) / 3;
                const int key = b < 8 ? GT_KEY_DEALER : (int)(b - 8 - 3 * q);
                block(key, b < 8 ? grp * 8 + b : grp, op, b < 8 ? 0 : 1 + q, D);
                if (b < 8) {
                    const u64 beta = D[5] & 1;
                    mat[b] = D[1]; mat[8 + b] = D[2]; mat[16 + b] = D[0] - D[1] - D[2];
                    mat[24 + b] = D[3]; mat[32 + b] = D[4]; mat[40 + b] = D[0] ^ D[3] ^ D[4];
                    mat[48 + b] = D[6]; mat[56 + b] = D[7]; mat[64 + b] = beta - D[6] - D[7];
                    const u32 b0_ = (u32)(D[5] >> 1) & 1, b1_ = (u32)(D[5] >> 2) & 1;
                    mat[72 + b] = b0_ | (b1_ << 1) | ((((u32)beta ^ b0_ ^ b1_) & 1) << 2);
                } else {
#pragma unroll
                    for (int s = 0; s < 8; s++) mat[80 + (b - 8) * 8 + s] = D[s];
                }
            }
        }
        __syncthreads();
        const Sh one1 = pub(p, 1);
        for (u32 s0 = 0; s0 < 8; s0 += ncol) {
            const u32 sl = s0 + cl, s = sl < 8 ? sl : 7;
            const bool mine = active && sl < 8, act = mine && s < live();
            Dealer D;
            D.rA.o = mat[p * 8 + s]; D.rA.n = mat[pn * 8 + s]; D.rho.o = mat[24 + p * 8 + s]; D.rho.n = mat[24 + pn * 8 + s];
            D.bA.o = mat[48 + p * 8 + s]; D.bA.n = mat[48 + pn * 8 + s];
            D.bBo = (u32)(mat[72 + s] >> p) & 1; D.bBn = (u32)(mat[72 + s] >> pn) & 1;
            const u64 AG = mat[80 + p * 8 + s] ^ mat[80 + pn * 8 + s], AE = mat[104 + p * 8 + s] ^ mat[104 + pn * 8 + s];
            const Sh v = { value(2, p, 0, s) - value(1, p, 0, s), value(2, p, 1, s) - value(1, p, 1, s) };
            const Sh bit = b2a(W, p, not_bit(p, ge_bit_masks(W, p, v, D, AG, AE, act)), D, act);
            if (mine && W.real) {
                value(0, p, 0, s) = 2 * value(0, p, 0, s) + bit.o + one1.o;
                value(0, p, 1, s) = 2 * value(0, p, 1, s) + bit.n + one1.n;
            }
        }
    }
};

// Four wavefronts per workgroup: at most one workgroup per compute unit, a wavefront has all registers of its SIMD; with one or
// two the registers are cut for two wavefronts per SIMD (70 spill, 107 with thresholds).
// Bound: a large batch by the vector ALU (see k_eqgrid), a small one by the chain of an access: three
// PRF blocks one after the other, nine rounds, three barriers.  Measured, with one party per wavefront and a barrier per
// message, in workgroups of four, now: 10^6 instances x 64 features, depth 10, 46.6, 34.5, 27 ms;
// 16 trees of depth 5 on 5,003 x 30 with thresholds 0.74, 0.58, 0.46 ms; 10^4 x 16, depth
// 7, thresholds 0.26 -> 0.16 ms; one instance 153 -> 127 us.  For NW see infer_shape.
template <bool THR, int NW>
__global__ __launch_bounds__(64 * NW, NW == 4 ? 1 : 2) void k_infer(InferArgs a)
{
    __shared__ uint4 s_msg[NW][GT_WMSG_QUADS];
    __shared__ u64 s_rows[NW][GT_EQ_ROWS];
    __shared__ u64 s_cnt[NW][6];
    __shared__ u64 s_mat[GT_INFER_OCT(NW)][GT_INFER_MAT];
    __shared__ u64 s_val[GT_INFER_OCT(NW)][3 * GT_INFER_VAL];
    __shared__ u64 s_sum[GT_INFER_OCT(NW)][48];
    const u32 wave = __builtin_amdgcn_readfirstlane(threadIdx.x / GT_LANES);
    InferWg<NW == 4 ? PRF_ALONE : PRF_PAIR_LOOP> X;
    X.E.init(a.c.keys, s_msg[wave], s_rows[wave], s_cnt[wave]);
    WWire &W = X.E.W;
    X.p = W.p; X.pn = W.pn; X.keys = a.c.keys;
    X.ncol = GT_INFER_LANES(NW) / a.noct;
    const u32 q = wave * GT_TP + W.t, o = q % a.noct;
    X.cl = q / a.noct; X.active = X.cl < X.ncol; X.one = X.cl == 0 && W.real;
    X.mat = s_mat[o]; X.val = s_val[o]; X.sum = s_sum[o];
    X.ngrp = a.N8 / 8; X.NI = a.NI;
    const Sh one = pub(W.p, 1);
    const int p = W.p;
    const u32 S = THR ? 3 : 2;
    const u64 ntile = (X.ngrp + a.noct - 1) / a.noct, nleaf = (u64)1 << a.H, nint = nleaf - 1;
    for (u64 item = blockIdx.x; item < ntile * a.ntrees; item += gridDim.x) {
        const u64 tree = item / ntile, tile = item % ntile;
        const u32 op0 = a.c.op + (u32)tree * (a.H * S + 1);
        X.grp = tile * a.noct + o;
        __syncthreads();
        if (X.one) {
#pragma unroll
            for (int s = 0; s < 8; s++) { X.value(0, p, 0, s) = 0; X.value(0, p, 1, s) = 0; }
        }
        for (u32 n = 0; n <= a.H; n++) {
            // level n's ids (and thresholds) at the index; after the last level the labels
            const bool labels = n == a.H;
            const u64 base = ((u64)1 << n) - 1, off = labels ? tree * nleaf : tree * nint + base;
            u64 zo[8], zn[8], yo[8], yn[8];
            X.template access<false, THR ? 2 : 1>(op0 + n * S, 0, base, 1u << n, labels ? a.leaf : a.feat, a.thr, off, THR && !labels, a.I, a.d,
                                                  zo, zn, yo, yn);
            if (labels) {
                if (X.one) {
#pragma unroll
                    for (int s = 0; s < 8; s++)
                        if (X.grp * 8 + s < a.NI) { const Sh z = { zo[s], zn[s] }; st(a.out, p, tree * a.NI + X.grp * 8 + s, z); }
                }
                break;
            }
            if (X.one) {
#pragma unroll
                for (int s = 0; s < 8; s++) {
                    X.value(1, p, 0, s) = zo[s]; X.value(1, p, 1, s) = zn[s];
                    if (THR) { X.value(2, p, 0, s) = yo[s]; X.value(2, p, 1, s) = yn[s]; }
                }
            }
            X.template access<true, 1>(op0 + n * S + 1, 1, 0, a.d, a.feat, a.feat, 0, false, a.I, a.d, zo, zn, yo, yn);
            if (X.one) {
#pragma unroll
                for (int s = 0; s < 8; s++) {
                    if (THR) { X.value(1, p, 0, s) = zo[s]; X.value(1, p, 1, s) = zn[s]; }
                    else {
                        X.value(0, p, 0, s) = 2 * X.value(0, p, 0, s) + zo[s] + one.o;
                        X.value(0, p, 1, s) = 2 * X.value(0, p, 1, s) + zn[s] + one.n;
                    }
                }
            }
            if (THR) X.greater(op0 + n * S + 2);
        }
        W.drain();
    }
    W.flush(a.c.wire);
}
