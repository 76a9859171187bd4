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
    u32 noct;                  // groups of 8 instances per tile, at most GT_INFER_OCT(NW), GT_AHEAD_OCT(NQ)
    u32 cus;                   // compute units of the device
};

// k_infer: a workgroup is NW wavefronts (1; 2 or 4 for some tiles that the caller asks for), each with the three parties in 21 lanes (WWire).  Its 21 NW lanes per party are
// split into noct groups of 8 instances x ncol columns: lane (o, cl) tests the 8 instances of group o against columns cl,
// cl + ncol, ... of the current access and adds up its share of the inner products in registers; the ncol partial
// sums meet in LDS.  The messages of the tests stay inside a wavefront; a workgroup synchronises three times per
// access, where the offline and zero-sharing words of the rows, evaluated by all lanes side by side, and the sums
// change hands.  k_infer_ahead, for few instances, is described further down.
// words per group of 8 instances.  Material of an access: r's arithmetic and Boolean components
// [6][8], zero-sharing words [2 streams, one without thresholds][3 keys][8]; of a comparison: [9][8] components (r, r's bits,
// beta), beta's bits [8], mask words [2][3][8].  Sums: [2, 1][3][8].  Values: index, id, threshold by component, [3][8]
// each: a component is written by the party whose own it is.
// The material's stride is 2 words modulo 32, so that the groups' and the parties' words of a step lie in different banks.
#define GT_INFER_MAT(THR) ((THR) ? 130 : 98)           // 128 and 72 used
#define GT_INFER_SUM(THR) ((THR) ? 48 : 24)
#define GT_INFER_VAL 24

// Adds up what the lanes of a wavefront hold for the same group of instances (lanes t, t + noct, .. of a party; q0: number of
// the wavefront's first lane in the workgroup's party) and adds the sums to sum[group * stride + 8 party ..]; a lane
// that is not `active` holds nothing.  Every lane adds its words by itself; with a single group (staged), where 21 lanes would meet
// at every word (one instance alone: 4,000 cycles an access), the lanes' words go through `stage` (8 * GT_LANES words) and
// an output is two lanes' work.  1,847 trees of depth 5 on one instance of 15 features 111 us by atomic adds, 98 through LDS, 50,000 x 294,
// depth 6, 1.45 and 1.43 ms.  Not with two groups (208,758 x 200, depth 3: 1.98 and 2.01 ms) or thresholds: while the lanes held the rows'
// opened values, 148 registers spilled for 101 (1.59 and 1.77 ms with one group of the 50,000 x 294, 37,015 x 47, depth 6, two groups 428 and 484 us); now
// 52 would for 17, and 1,847 trees on one instance with thresholds would take 106 us for 129.
template <bool STAGED>
__device__ __forceinline__ void group_sums(const WWire &W, u64 *stage, const u64 (&acc)[8], bool active, u32 q0, u32 noct, u64 *sum, u32 stride)
{
    if (!STAGED) {
        u64 *d = sum + (q0 + W.t) % noct * stride + W.p * 8;
        if (active && W.real) {
#pragma unroll
            for (int s = 0; s < 8; s++) atomicAdd((unsigned long long *)&d[s], (unsigned long long)acc[s]);
        }
        return;
    }
    wave_sync();
    ulonglong2 *out = (ulonglong2 *)(stage + W.m * 8);
#pragma unroll
    for (int j = 0; j < 4; j++) out[j] = make_ulonglong2(active ? acc[2 * j] : 0, active ? acc[2 * j + 1] : 0);
    wave_sync();
    const u64 *in = stage + W.p * GT_TP * 8;
    const u32 t0 = W.t >> 3, s = W.t & 7;              // 16 halves of the eight outputs
    u64 v = 0;
    for (u32 t = t0; t < GT_TP; t += 8) {              // four loads in flight
        u64 x[4];
#pragma unroll
        for (int j = 0; j < 4; j++) x[j] = in[(t + j * 2 < GT_TP ? t + j * 2 : t0) * 8 + s];
#pragma unroll
        for (int j = 0; j < 4; j++) v += t + j * 2 < GT_TP ? x[j] : 0;
    }
    if (W.real && W.t < 16) atomicAdd((unsigned long long *)&sum[W.p * 8 + s], (unsigned long long)v);
}

template <int ISSUE, bool STAGED>
struct InferWg {
    EqWave E;
    u64 *sums;                   // of the workgroup's groups
    u64 *opened;                 // this wavefront's copy of the group's opened values u + r - base, 8 words
    u64 *mat, *val, *sum;        // of this lane's group: material, values, sums
    const u32 *keys;
    u32 cl, ncol, q0, noct, stride;      // q0: the wavefront's first lane in the workgroup's party
    u64 ngrp, grp, NI;           // groups of the batch, this lane's group
    bool active, one;            // the lane has a group / is the one that counts and stores for its group and party
    int p, pn;

    // component `comp` of a value, for both parties that hold it
    __device__ __forceinline__ u64 &value(int which, int comp, int s) { return val[which * GT_INFER_VAL + comp * 8 + s]; }
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
        {
            u64 snd[8], mn[8], rcv[8];
#pragma unroll
            for (int s = 0; s < 8; s++) {
                snd[s] = value(which, p, s) + mat[p * 8 + s]; mn[s] = value(which, pn, s) + mat[W.pn * 8 + s];
            }
            W.open64<8>(snd, rcv);
            W.nopen += one ? 64u * live() : 0u;
            // every lane of a group has the same words; kept in LDS, like r's Boolean components, for the access's steps
#pragma unroll
            for (int s = 0; s < 8; s++) opened[s] = snd[s] + mn[s] + rcv[s] - base;
            wave_sync();
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
            const u32 f = E.template tests<false, ISSUE>(op, (u64)col * ngrp + grp, [&](int h, u64 (&cd)[4], u64 (&ro)[4], u64 (&rn)[4]) {
#pragma unroll
                for (int j = 0; j < 4; j++) {
                    cd[j] = opened[h + j] - col; ro[j] = mat[24 + p * 8 + h + j]; rn[j] = mat[24 + W.pn * 8 + h + j];
                }
            }, 0, 0, act ? live() : 0u, [&]() {
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
        group_sums<STAGED>(W, E.rows, acc, active, q0, noct, sums, stride);
        if (NDOT == 2 && nd2) group_sums<STAGED>(W, E.rows, acc2, active, q0, noct, sums + 24, stride);
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
            const Sh v = { value(2, p, s) - value(1, p, s), value(2, pn, s) - value(1, pn, s) };
            const Sh bit = b2a(W, p, not_bit(p, ge_bit_masks(W, p, v, D, AG, AE, act)), D, act);
            if (mine && W.real) value(0, p, s) = 2 * value(0, p, s) + bit.o + one1.o;
        }
    }
};

// Bound: the vector ALU (see k_eqgrid).  The registers are cut for two wavefronts per SIMD: 9 to 13 spill, 14 to 17 with thresholds, since the rows'
// opened values and Boolean components are read from LDS in every step (68 and 101 when the lanes held them: 16 trees of depth 5 on
// 5,003 x 30 with thresholds 439 us, 414 now; 300,000 x 20, depth 5, 1,055 and 1,006; 10^6 x 64, depth 10, 26.9 and 26.7 ms).  Three wavefronts of
// 168 registers spill 100 around the accesses, which only accesses of thousands of columns outweigh: 50,000 x 294, depth 6, 1.66 and 2.53 ms.
// Before, with one party per wavefront and a barrier per message, and in workgroups of four wavefronts: 10^6 x 64 46.6 and 34.5 ms,
// 16 trees 0.74 and 0.58 ms.  For NW see infer_shape.
template <bool THR, int NW, bool STAGED>
__global__ __launch_bounds__(64 * NW, 2) void k_infer(InferArgs a)
{
    __shared__ uint4 s_msg[NW][GT_WMSG_QUADS];
    __shared__ u64 s_rows[NW][GT_EQ_ROWS];
    __shared__ u64 s_cnt[NW][6];
    __shared__ u64 s_mat[GT_INFER_OCT(NW)][GT_INFER_MAT(THR)];
    __shared__ u64 s_val[GT_INFER_OCT(NW)][(THR ? 3 : 2) * GT_INFER_VAL];
    __shared__ u64 s_sum[GT_INFER_OCT(NW)][GT_INFER_SUM(THR)];
    __shared__ u64 s_open[NW][GT_INFER_OCT(NW)][8];
    __shared__ __align__(16) u32 s_keys[40];               // the five keys: the blocks of the rows are evaluated with one or another by lane
    static_assert(sizeof s_msg + sizeof s_rows + sizeof s_cnt + sizeof s_mat + sizeof s_val + sizeof s_sum + sizeof s_open + sizeof s_keys <= NW * 20480,
                  "eight wavefronts on a compute unit's 160 KB");
    const u32 wave = __builtin_amdgcn_readfirstlane(threadIdx.x / GT_LANES);
    InferWg<PRF_PAIR_LOOP, STAGED> X;
    X.E.init(a.c.keys, s_msg[wave], s_rows[wave], s_cnt[wave]);
    WWire &W = X.E.W;
    X.p = W.p; X.pn = W.pn; X.keys = s_keys;
    if (threadIdx.x < 40) s_keys[threadIdx.x] = a.c.keys[threadIdx.x];          // read after the first item's barrier
    X.ncol = GT_INFER_LANES(NW) / a.noct;
    const u32 q = wave * GT_TP + W.t, o = q % a.noct;
    X.cl = q / a.noct; X.active = X.cl < X.ncol; X.one = X.cl == 0 && W.real;
    X.sums = s_sum[0]; X.stride = GT_INFER_SUM(THR); X.q0 = wave * GT_TP; X.noct = a.noct;
    X.opened = s_open[wave][o]; X.mat = s_mat[o]; X.val = s_val[o]; X.sum = s_sum[o];
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
            for (int s = 0; s < 8; s++) X.value(0, p, s) = 0;
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
                    X.value(1, p, s) = zo[s];
                    if (THR) X.value(2, p, s) = yo[s];
                }
            }
            X.template access<true, 1>(op0 + n * S + 1, 1, 0, a.d, a.feat, a.feat, 0, false, a.I, a.d, zo, zn, yo, yn);
            if (X.one) {
#pragma unroll
                for (int s = 0; s < 8; s++) {
                    if (THR) X.value(1, p, s) = zo[s];
                    else X.value(0, p, s) = 2 * X.value(0, p, s) + zo[s] + one.o;
                }
            }
            if (THR) X.greater(op0 + n * S + 2);
        }
        W.drain();
    }
    W.flush(a.c.wire);
}

// ---------------------------------------------------------------------------------
// Few instances: all workgroups at once on the chip, four wavefronts per SIMD at most, where the chain of a tile's
// accesses is all that counts.  4 NQ wavefronts (NQ = 4, 2 or 1).  2 NQ run the protocol: wavefronts w and w + NQ have the 21 lanes
// per party number w of the tile's 21 NQ, split into noct groups of 8 instances x ncol columns as in k_infer, the first on
// the instances 0-3 of a group, the other on 4-7.  The others evaluate all PRF blocks one interval ahead, because no
// block depends on anything but public indices: NQ the mask words and the rows' material, NQ the daBits.  A barrier ends an
// interval: {the sums of the access before, the opening of the next one}, then one per step, one per comparison.
// The PRF side of an interval:
//   opening            the first step's mask words
//   a step             the next step's mask words and daBits; in an access's last step the rows' material
//                      of what follows (access or comparison) and the daBits of the next access's first step
//   a comparison       the rows' material of the next level's access
// Every lane of a group computes the group's results, so that a result goes into the next opening without
// a barrier; sums are cleared in the opening that follows their last reading.
// Bound: the intervals' longer side, about 2,500 cycles of a PRF block and its handing over or of a step's rounds; on a full
// chip the vector ALU (masks and daBits of the columns that a level does not have are evaluated all the same).  Measured, in one
// wavefront per 21 lanes that did both, four per tile, and now: one instance of 22 features, depth 7, thresholds 127 -> 60 us;
// 10^4 x 16, depth 7, thresholds 161 -> 112 us; 300 x 100, depth 5, 89 -> 48 us; 1,000 trees of depth 3 on one instance 73 -> 44 us.
// Both sides on eight tests a lane, with two wavefronts per SIMD: 70, 104, 54 us for the first three.  The 128 registers of four
// wavefronts per SIMD spill 31 or 32, with thresholds 42 (128 to 172 bytes a lane).
#define GT_AHEAD_T 96                                  // words per group: material of an access to the tree, [6][8] and [2][3][8]
#define GT_AHEAD_F 72                                  // to the features, [6][8] and [3][8]
#define GT_AHEAD_G 128                                 // of a comparison, as in InferWg
// daBit rows test after test here, as the wavefronts of a half take them (in the order of eq_row one instance takes 60.1 us instead of 59.5)
#define GT_AHEAD_COMP (9 * (GT_TP + 1))
struct AheadStep { uint4 mask[4 * GT_LANES]; u64 rows[3 * GT_AHEAD_COMP]; u32 bits[GT_LANES]; };   // a step's material of 21 lanes per party

// The AND rounds of four equality tests, as EqWave::rounds for eight: [cd == 0] of tests 4h .. 4h + 3; the opened f has test j in
// bit 8 j, and so has bw, the Boolean components of the daBits.
__device__ __forceinline__ u32 eq_rounds4(WWire &W, u32 M0, u32 M2, const u64 (&A)[4], const u64 (&An)[4], u32 bw, const u64 (&cd)[4],
                                          const u64 (&rho_o)[4], const u64 (&rho_n)[4], u32 nl)
{
    u32 Ah[4], xo[4], xn[4];
#pragma unroll
    for (int s = 0; s < 4; s++) {                      // round 0, width 32
        const u32 dl = (u32)cd[s], dh = (u32)(cd[s] >> 32);
        const u32 tol = logic3<0xd2>((u32)rho_o[s], dl, M0), toh = logic3<0xd2>((u32)(rho_o[s] >> 32), dh, M0);
        const u32 tnl = logic3<0xd2>((u32)rho_n[s], dl, M2), tnh = logic3<0xd2>((u32)(rho_n[s] >> 32), dh, M2);
        xo[s] = xor3l(and3l(tol, tnl, toh, tnh), (u32)A[s], (u32)An[s]);
        Ah[s] = (u32)(A[s] >> 32) ^ (u32)(An[s] >> 32);
    }
    W.reshare<4>(xo, xn);
    u32 Po[2], Pn[2], H[2];
#pragma unroll
    for (int j = 0; j < 2; j++) {                      // round 1, width 16
        const u32 al = __builtin_amdgcn_perm(xo[2 * j + 1], xo[2 * j], 0x05040100u), ah = __builtin_amdgcn_perm(xo[2 * j + 1], xo[2 * j], 0x07060302u);
        const u32 bl = __builtin_amdgcn_perm(xn[2 * j + 1], xn[2 * j], 0x05040100u), bh = __builtin_amdgcn_perm(xn[2 * j + 1], xn[2 * j], 0x07060302u);
        Po[j] = and3l(al, bl, ah, bh) ^ __builtin_amdgcn_perm(Ah[2 * j + 1], Ah[2 * j], 0x05040100u);
        H[j] = __builtin_amdgcn_perm(Ah[2 * j + 1], Ah[2 * j], 0x07060302u);
    }
    W.reshare<2>(Po, Pn);
    u32 Q[1], Qn[1];                                   // round 2, width 8: test j in byte j from here on
    Q[0] = and3l(__builtin_amdgcn_perm(Po[1], Po[0], 0x06040200u), __builtin_amdgcn_perm(Pn[1], Pn[0], 0x06040200u),
                 __builtin_amdgcn_perm(Po[1], Po[0], 0x07050301u), __builtin_amdgcn_perm(Pn[1], Pn[0], 0x07050301u))
           ^ __builtin_amdgcn_perm(H[1], H[0], 0x06040200u);
    const u32 B = __builtin_amdgcn_perm(H[1], H[0], 0x07050301u);        // bits 56-63 of the mask words
    W.reshare<1>(Q, Qn);
    u32 R[1], Rn[1];                                   // rounds 3, 4, 5: widths 4, 2, 1
    R[0] = logic3<0x60>(0x0f0f0f0fu, and3l(Q[0], Qn[0], Q[0] >> 4, Qn[0] >> 4), B);
    W.reshare<1>(R, Rn);
    u32 S[1], Sn[1];
    S[0] = logic3<0x60>(0x03030303u, and3l(R[0], Rn[0], R[0] >> 2, Rn[0] >> 2), B >> 4);
    W.reshare<1>(S, Sn);
    u32 T[1], Tn[1];
    T[0] = logic3<0x60>(0x01010101u, and3l(S[0], Sn[0], S[0] >> 1, Sn[0] >> 1), B >> 6);
    W.reshare<1>(T, Tn);
    u32 fo[1] = { (T[0] ^ (bw >> W.p)) & 0x01010101u }, fr[1];           // bit -> arithmetic: open s xor beta
    W.pass<1>(fo, fr, W.pv);
    W.nopen += nl; W.nresh += 63u * nl;
    return xor3l(fo[0], Tn[0] ^ (bw >> W.pn), fr[0]);
}

template <bool THR, int NQ>
__global__ __launch_bounds__(256 * NQ, 4) void k_infer_ahead(InferArgs a)
{
    constexpr int OCT = GT_AHEAD_OCT(NQ);
    __shared__ uint4 s_msg[2 * NQ][2 * GT_LANES];
    __shared__ AheadStep s_step[2][NQ];
    __shared__ u64 s_matT[OCT][GT_AHEAD_T], s_matF[OCT][GT_AHEAD_F], s_matG[THR ? OCT : 1][GT_AHEAD_G];
    __shared__ u64 s_val[2][OCT][2 * GT_INFER_VAL];                // the index, of even and of odd levels
    __shared__ u64 s_th[THR ? OCT : 1][2 * GT_INFER_VAL];          // the threshold
    __shared__ u64 s_sumT[OCT][48], s_sumF[OCT][24];
    __shared__ u64 s_cnt[2 * NQ][6];
    // A workgroup's wavefronts go to the SIMDs in turn; the roles of the second, third, .. workgroup of a compute unit are
    // shifted, so that no SIMD gets the PRF wavefronts of all of them (300 trees on 30 x 50: 112 -> 93 us)
    const u32 wv = __builtin_amdgcn_readfirstlane(threadIdx.x / GT_LANES + (NQ < 4 ? NQ * (blockIdx.x / a.cus) : 0)) % (4 * NQ), wave = wv % NQ, half = wv / NQ & 1, h4 = 4 * half;
    const u32 ncol = GT_INFER_LANES(NQ) / a.noct, S = THR ? 3 : 2;
    const u64 ngrp = a.N8 / 8, ntile = (ngrp + a.noct - 1) / a.noct, tree = blockIdx.x / ntile, grp0 = (blockIdx.x % ntile) * a.noct;
    const u32 op0 = a.c.op + (u32)tree * (a.H * S + 1);
    u32 turn = 0;                                                        // steps so far: their material alternates between two buffers

    // The two sides run the same intervals: levels, steps and comparisons are public.
    if (wv >= 2 * NQ) {
        // ---- PRF: half 0 the masks and the rows, half 1 the daBits
        EqWave E;
        E.init(a.c.keys, nullptr, nullptr, nullptr);
        const WWire &W = E.W;
        const u32 q = wave * GT_TP + W.t, cl = q / a.noct;
        const u64 grp = grp0 + q % a.noct;
        // material of the rows of all groups: roles of a group 0-7 the dealer's blocks, then the words of streams st0, st0 + 1, ..
        // under the three keys; conv: with the components of a daBit
        const auto deal_rows = [&](u32 op, u64 *mat, u32 stride, u32 nstr, u32 st0, bool conv) {
            const u32 nroles = 8 + 3 * nstr;
            for (u32 r = wave * GT_LANES + (threadIdx.x & (GT_LANES - 1)); r < a.noct * nroles; r += NQ * GT_LANES) {
                const u32 g = r % a.noct, b = r / a.noct, i = (b - 8) / 3;
                if (grp0 + g >= ngrp) continue;
                u64 *m = mat + g * stride, D[8];
                const int key = b < 8 ? GT_KEY_DEALER : (int)(b - 8 - 3 * i);
                Key kv;
#pragma unroll
                for (int j = 0; j < 8; j++) kv.k[j] = a.c.keys[key * 8 + j];
                chacha8<PRF_PAIR>(kv, b < 8 ? (grp0 + g) * 8 + b : grp0 + g, op, b < 8 ? 0 : st0 + i, D);
                if (b < 8) {
                    m[b] = D[1]; m[8 + b] = D[2]; m[16 + b] = D[0] - D[1] - D[2];
                    m[24 + b] = D[3]; m[32 + b] = D[4]; m[40 + b] = D[0] ^ D[3] ^ D[4];
                    if (conv) {
                        const u64 beta = D[5] & 1;
                        const u32 b0 = (u32)(D[5] >> 1) & 1, b1 = (u32)(D[5] >> 2) & 1;
                        m[48 + b] = D[6]; m[56 + b] = D[7]; m[64 + b] = beta - D[6] - D[7];
                        m[72 + b] = b0 | (b1 << 1) | ((((u32)beta ^ b0 ^ b1) & 1) << 2);
                    }
                } else {
                    m += (conv ? 80 : 48) + (b - 8) * 8;
#pragma unroll
                    for (int s = 0; s < 8; s++) m[s] = D[s];
                }
            }
        };
        const auto deal_mask = [&](u32 op, u32 k0, u32 at) {
            u64 A[8];
            chacha8<PRF_PAIR>(E.own, (u64)(k0 + cl) * ngrp + grp, op, 1, A);
            uint4 *m = s_step[at & 1][wave].mask + W.m;
#pragma unroll
            for (int j = 0; j < 4; j++)
                m[j * GT_LANES] = make_uint4((u32)A[2 * j], (u32)(A[2 * j] >> 32), (u32)A[2 * j + 1], (u32)(A[2 * j + 1] >> 32));
        };
        const auto deal_bits = [&](u32 op, u32 k0, u32 at) {
            AheadStep &T = s_step[at & 1][wave];
            T.bits[W.m] = E.template deal_bits<PRF_PAIR, GT_AHEAD_COMP, GT_TP + 1, 3 * (GT_TP + 1)>(op, (u64)(k0 + cl) * ngrp + grp, T.rows + W.t);
        };
        // the steps of an access after its first: their material, then the interval of the step before
        const auto deal_steps = [&](u32 op, u32 w) {
            for (u32 k0 = ncol; k0 < w; k0 += ncol) {
                turn++;
                if (half == 0) deal_mask(op, k0, turn); else deal_bits(op, k0, turn);
                __syncthreads();
            }
            turn++;
        };
        if (half == 0) deal_rows(op0, s_matT[0], GT_AHEAD_T, THR && a.H > 0 ? 2 : 1, 2, false); else deal_bits(op0, 0, 0);
        __syncthreads();
        for (u32 n = 0; n <= a.H; n++) {
            const u32 opT = op0 + n * S, opF = opT + 1;
            if (half == 0) deal_mask(opT, 0, turn);
            __syncthreads();
            deal_steps(opT, 1u << n);
            if (n < a.H) { if (half == 0) deal_rows(opF, s_matF[0], GT_AHEAD_F, 1, 2, false); else deal_bits(opF, 0, turn); }
            __syncthreads();
            if (n == a.H) break;
            if (half == 0) deal_mask(opF, 0, turn);
            __syncthreads();
            deal_steps(opF, a.d);
            if (half == 1) deal_bits(opT + S, 0, turn);
            if (THR) {
                if (half == 0) deal_rows(opF + 1, s_matG[0], GT_AHEAD_G, 2, 1, true);
                __syncthreads();
            }
            if (half == 0) deal_rows(opT + S, s_matT[0], GT_AHEAD_T, THR && n + 1 < a.H ? 2 : 1, 2, false);
            __syncthreads();
        }
        return;
    }

    // ---- the protocol
    WWire W;
    W.init(s_msg[wv], s_cnt[wv]);
    const int p = W.p, pn = W.pn;
    const u32 M0 = p == 0 ? ~0u : 0u, M2 = p == 2 ? ~0u : 0u;
    const u32 q = wave * GT_TP + W.t, o = q % a.noct, cl = q / a.noct;
    const bool active = cl < ncol, first = cl == 0 && W.real;           // first: counts and stores for its instances and party
    const u64 grp = grp0 + o, i0 = grp * 8 + h4, nleaf = (u64)1 << a.H, nint = nleaf - 1;
    const u32 live8_ = grp < ngrp ? live8(grp * 8, a.NI) : 0u, live = live8_ <= h4 ? 0u : (live8_ - h4 < 4 ? live8_ - h4 : 4u);
    const Sh one = pub(p, 1);
    const u32 k1o = (u32)one.o + 1, k1n = (u32)one.n + 1;
    u64 *const matT = s_matT[o], *const matF = s_matF[o], *const sumT = s_sumT[o], *const sumF = s_sumF[o];
    u64 uo[4], un[4], cpub[4], rho_o[4], rho_n[4], acc[4], acc2[4];
    const u32 own8 = p * 8 + h4, nxt8 = pn * 8 + h4;                    // the lane's first word of the party's own / next eight
    const u32 vo = p * 16 + h4, vn = vo + 8;                            // ... in a value: [party][own, next][8]
    // the group's result of an access: sums, the party's zero-sharing words, one reshare round
    const auto result = [&](const u64 *sum, const u64 *words, u64 (&zo)[4], u64 (&zn)[4]) {
#pragma unroll
        for (int s = 0; s < 4; s++) zo[s] = sum[own8 + s] + (words[own8 + s] - words[nxt8 + s]);
        W.reshare64<4>(zo, zn);
        W.nresh += first ? 64u * live : 0u;
    };
    // the opening of an access: c = u + r - base, public afterwards
    const auto open_access = [&](const u64 *mat, u64 base) {
        u64 snd[4], mn[4], rcv[4];
#pragma unroll
        for (int s = 0; s < 4; s++) {
            snd[s] = uo[s] + mat[own8 + s]; mn[s] = un[s] + mat[nxt8 + s];
            rho_o[s] = mat[24 + own8 + s]; rho_n[s] = mat[24 + nxt8 + s];
        }
        W.open64<4>(snd, rcv);
#pragma unroll
        for (int s = 0; s < 4; s++) { cpub[s] = snd[s] + mn[s] + rcv[s] - base - cl; acc[s] = 0; acc2[s] = 0; }
        W.nopen += first ? 64u * live : 0u;
    };
    // one step: the opened bits of the tests of columns k0 + cl; the daBits' arithmetic components of test s are
    // bit(p, s), bit(pn, s)
    const auto rounds = [&](u32 k0, bool act) -> u32 {
        const AheadStep &T = s_step[turn & 1][wave];
        u64 A[4], An[4], cd[4];
#pragma unroll
        for (int j = 0; j < 2; j++) {
            const uint4 v = T.mask[(h4 / 2 + j) * GT_LANES + W.m], w = T.mask[(h4 / 2 + j) * GT_LANES + W.nx];
            A[2 * j] = (u64)v.x | ((u64)v.y << 32); A[2 * j + 1] = (u64)v.z | ((u64)v.w << 32);
            An[2 * j] = (u64)w.x | ((u64)w.y << 32); An[2 * j + 1] = (u64)w.z | ((u64)w.w << 32);
        }
        const u32 bw = (T.bits[W.m] | T.bits[W.nx] | T.bits[W.pv]) >> h4;
#pragma unroll
        for (int s = 0; s < 4; s++) cd[s] = cpub[s] - k0;
        return eq_rounds4(W, M0, M2, A, An, bw, cd, rho_o, rho_n, act ? live : 0u);
    };
    // one product per word: with the component's stride of its own (c * 198 + ..) 10^4 x 16, depth 7, thresholds takes 114.0 us, 113.3 so
    const auto bit = [&](int c, int s) { return s_step[turn & 1][wave].rows[(c * 9 + h4 + s) * (GT_TP + 1) + W.t]; };
    // adds up the four words of a group's lanes: every lane by itself, or with one or two groups, where 10 to 21 lanes would meet at
    // every word, through the message region (one instance: 4,000 cycles an access without that)
    const auto add_up = [&](const u64 (&x)[4], u64 *sum, u32 stride) {
        if (a.noct > 2) {
            if (active && W.real) {
#pragma unroll
                for (int s = 0; s < 4; s++) atomicAdd((unsigned long long *)&sum[o * stride + own8 + s], (unsigned long long)x[s]);
            }
            return;
        }
        u64 *stage = (u64 *)W.buf;
        wave_sync();
        ulonglong2 *out = (ulonglong2 *)(stage + W.m * 4);
        out[0] = make_ulonglong2(active ? x[0] : 0, active ? x[1] : 0);
        out[1] = make_ulonglong2(active ? x[2] : 0, active ? x[3] : 0);
        wave_sync();
        const u32 step = a.noct == 1 ? 5 : 4, t0 = W.t >> 2, s = W.t & 3;        // 20 or 16 lanes, each the words of every 5th or 4th lane
        const u64 *in = stage + p * GT_TP * 4 + s;
        u64 v = 0, y[6];
#pragma unroll
        for (int j = 0; j < 6; j++) y[j] = in[(t0 + j * step < GT_TP ? t0 + j * step : t0) * 4];
#pragma unroll
        for (int j = 0; j < 6; j++) v += t0 + j * step < GT_TP ? y[j] : 0;
        if (W.real && t0 < step) atomicAdd((unsigned long long *)&sum[(wave * GT_TP + t0) % a.noct * stride + own8 + s], (unsigned long long)v);
    };

    __syncthreads();
    for (u32 n = 0; n <= a.H; n++) {
        // level n's ids (and thresholds) at the index; after the last level the labels
        const bool labels = n == a.H, two = THR && !labels;
        const u64 base = ((u64)1 << n) - 1, off = labels ? tree * nleaf : tree * nint + base;
        const u32 w = 1u << n;
        const P6 &W1 = labels ? a.leaf : a.feat;
        if (n == 0) {
#pragma unroll
            for (int s = 0; s < 4; s++) { uo[s] = 0; un[s] = 0; }
        } else if (THR) {
#pragma unroll
            for (int s = 0; s < 4; s++) { uo[s] = s_val[n & 1][o][vo + s]; un[s] = s_val[n & 1][o][vn + s]; }
        } else {
            u64 zo[4], zn[4];
            result(sumF, matF + 48, zo, zn);
#pragma unroll
            for (int s = 0; s < 4; s++) {
                uo[s] = 2 * (n == 1 ? 0 : s_val[(n - 1) & 1][o][vo + s]) + zo[s] + one.o;
                un[s] = 2 * (n == 1 ? 0 : s_val[(n - 1) & 1][o][vn + s]) + zn[s] + one.n;
                if (first) { s_val[n & 1][o][vo + s] = uo[s]; s_val[n & 1][o][vn + s] = un[s]; }
            }
        }
        if (first) {
#pragma unroll
            for (int s = 0; s < 4; s++) { sumT[own8 + s] = 0; if (THR) sumT[24 + own8 + s] = 0; }
        }
        open_access(matT, base);
        __syncthreads();
        for (u32 k0 = 0; k0 < w; k0 += ncol, turn++) {
            const u32 col = k0 + cl;
            const bool act = active && col < w;
            Sh Wk = { 0, 0 }, Wk2 = { 0, 0 };
            if (act) Wk = ld(W1, p, off + col);
            if (act && two) Wk2 = ld(a.thr, p, off + col);
            const u32 f = rounds(k0, act);
            // columns beyond w: W = 0, the sum stays (see k_eqgrid)
            const u64 Ss = Wk.o + Wk.n, nc = ~(one.o * Ss + one.n * Wk.o);
            const u64 S2 = Wk2.o + Wk2.n, nc2 = ~(one.o * S2 + one.n * Wk2.o);
#pragma unroll
            for (int s = 0; s < 4; s++) {
                const u32 m = (u32)((int)(f << (31 - 8 * s)) >> 31);
                const u64 mm = (u64)m | ((u64)m << 32), bo = bit(p, s), bn = bit(pn, s);
                acc[s] += ((mm & nc) + bo * Ss + bn * Wk.o) ^ mm;
                if (THR) acc2[s] += ((mm & nc2) + bo * S2 + bn * Wk2.o) ^ mm;
            }
            if (k0 + ncol >= w) {
                add_up(acc, s_sumT[0], 48);
                if (THR && two) add_up(acc2, s_sumT[0] + 24, 48);
            }
            __syncthreads();
        }
        if (labels) break;
        // the instance's feature at the id
        result(sumT, matT + 48, uo, un);
        if (THR) {                                     // the thresholds, an instance per lane
            for (u32 s0 = 0; s0 < 4; s0 += ncol) {
                const u32 sl = s0 + cl, s = sl < 4 ? sl : 3;
                const bool mine = active && sl < 4;
                const u64 zo = sumT[24 + own8 + s] + (matT[72 + own8 + s] - matT[72 + nxt8 + s]);
                const u64 zn = W.reshare1(zo, mine && s < live ? 64u : 0u);
                if (mine && W.real) { s_th[o][vo + s] = zo; s_th[o][vn + s] = zn; }
            }
        }
        if (first) {
#pragma unroll
            for (int s = 0; s < 4; s++) sumF[own8 + s] = 0;
        }
        open_access(matF, 0);
        __syncthreads();
        const u64 *xpo = own_of(a.I, p), *xpn = nxt_of(a.I, p), lastrow = a.NI - 1;      // rows beyond the batch read its last one
        for (u32 k0 = 0; k0 < a.d; k0 += ncol, turn++) {
            const u32 col = k0 + cl, c = active && col < a.d ? col : a.d - 1;
            const bool act = active && col < a.d;
            u64 xo[4], xn[4];
#pragma unroll
            for (int s = 0; s < 4; s++) {
                const u64 i = i0 + s < lastrow ? i0 + s : lastrow;
                xo[s] = xpo[i * a.d + c]; xn[s] = xpn[i * a.d + c];
            }
            const u32 f = rounds(k0, act);
#pragma unroll
            for (int s = 0; s < 4; s++) {
                const u32 m = (u32)((int)(f << (31 - 8 * s)) >> 31);
                const Sh e = { eq_select(bit(p, s), m, k1o), eq_select(bit(pn, s), m, k1n) }, x = { xo[s], xn[s] };
                if (act) acc[s] += prod3(e, x);
            }
            if (k0 + ncol >= a.d) add_up(acc, s_sumF[0], 24);
            __syncthreads();
        }
        if (THR) {
            // index <- 2 index + [x > theta] + 1, an instance per lane
            const u64 *mat = s_matG[o];
            for (u32 s0 = 0; s0 < 4; s0 += ncol) {
                const u32 sl = s0 + cl, s = sl < 4 ? sl : 3;
                const bool mine = active && sl < 4, act = mine && s < live;
                const u32 so = own8 + s, sn = nxt8 + s;
                Sh x;
                x.o = sumF[so] + (matF[48 + so] - matF[48 + sn]);
                x.n = W.reshare1(x.o, act ? 64u : 0u);
                Dealer D;
                D.rA.o = mat[so]; D.rA.n = mat[sn]; D.rho.o = mat[24 + so]; D.rho.n = mat[24 + sn];
                D.bA.o = mat[48 + so]; D.bA.n = mat[48 + sn];
                D.bBo = (u32)(mat[72 + h4 + s] >> p) & 1; D.bBn = (u32)(mat[72 + h4 + s] >> pn) & 1;
                const u64 AG = mat[80 + so] ^ mat[80 + sn], AE = mat[104 + so] ^ mat[104 + sn];
                const Sh v = { s_th[o][vo + s] - x.o, s_th[o][vn + s] - x.n };
                const Sh b = b2a(W, p, not_bit(p, ge_bit_masks(W, p, v, D, AG, AE, act)), D, act);
                if (mine && W.real) {
                    s_val[(n + 1) & 1][o][vo + s] = 2 * (n == 0 ? 0 : s_val[n & 1][o][vo + s]) + b.o + one.o;
                    s_val[(n + 1) & 1][o][vn + s] = 2 * (n == 0 ? 0 : s_val[n & 1][o][vn + s]) + b.n + one.n;
                }
            }
            __syncthreads();
        }
    }
    u64 zo[4], zn[4];
    result(sumT, matT + 48, zo, zn);
    if (first) {
#pragma unroll
        for (int s = 0; s < 4; s++)
            if (i0 + s < a.NI) st(a.out, p, tree * a.NI + i0 + s, Sh{ zo[s], zn[s] });
    }
    W.flush(a.c.wire);
}
