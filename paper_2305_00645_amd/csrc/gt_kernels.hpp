// Kernels of the GTree hot path for gfx950.  See gt_device.hpp for the execution
// models (three parties per wavefront, or per workgroup; messages through LDS).
#pragma once
#include "gt_device.hpp"

#define GT_BLOCK dim3(GT_LANES, 3, 1)

// grid-stride loop over tiles of 64 elements; every lane of the workgroup runs the
// same number of iterations, so the barriers inside the protocols stay uniform
#define GT_FOR_TILES(n)                                                                    \
    for (u64 tile_ = blockIdx.x, ntiles_ = ((u64)(n) + GT_LANES - 1) / GT_LANES; tile_ < ntiles_; tile_ += gridDim.x)
#define GT_ELEM() (tile_ * GT_LANES + threadIdx.x)

// keys: the five keys; op: operation id; wire: the context's six message counters
// (payload bits sent by party p to its successor [2p] and to its predecessor [2p+1])
struct KCommon { const u32 *keys; u32 op; u64 *wire; };

// number of the lane's 8 consecutive elements (first one i0) that exist below n
__device__ __forceinline__ u32 live8(u64 i0, u64 n) { return i0 >= n ? 0u : (n - i0 >= 8 ? 8u : (u32)(n - i0)); }

// ---------------------------------------------------------------------------------
// A PRF block holds the words of 8 consecutive elements, one block per lane; memory wants
// consecutive elements in consecutive lanes.  The 512 words of a wavefront change hands through
// LDS: word s of lane l at s*72 + l, element 64 j + l of the tile in word l%8 of lane 8 j + l/8;
// neither the stores nor the loads meet bank conflicts.
#define GT_TR_WORDS (8 * 72)
__device__ __forceinline__ void tr_put(u64 *tr, u32 lane, const u64 (&w)[8])
{
#pragma unroll
    for (int s = 0; s < 8; s++) tr[s * 72 + lane] = w[s];
}
__device__ __forceinline__ u64 tr_get(const u64 *tr, u32 lane, int j) { return tr[(lane & 7) * 72 + 8 * j + (lane >> 3)]; }

// Share^A (Sec. II-B): x1, x2 from the owner's key (streams 0 and 1), x3 = x - x1 - x2.
// Bound: memory (one word read, six written).  2^24 words: 1.30 ms when every lane stored its own
// 8 consecutive words (a line per lane and instruction), 0.19 ms now (5.0 TB/s).
// put(e, a, b, x3) stores the three components of element e.
template <class F>
__device__ __forceinline__ void share_tiles(const u32 *keys, int key, u32 op, const u64 *plain, u64 n, u64 *ta, u64 *tb, F put)
{
    const Key ko = load_key(keys, key);
    const u32 lane = threadIdx.x & (GT_LANES - 1), wave = threadIdx.x / GT_LANES;
    for (u64 t = (u64)blockIdx.x * 4 + wave; t < (n + 511) / 512; t += (u64)gridDim.x * 4) {
        u64 w[8];
        wave_sync();
        chacha8(ko, t * GT_LANES + lane, op, 0, w);
        tr_put(ta, lane, w);
        chacha8(ko, t * GT_LANES + lane, op, 1, w);
        tr_put(tb, lane, w);
        wave_sync();
#pragma unroll
        for (int j = 0; j < 8; j++) {
            const u64 e = t * 512 + j * GT_LANES + lane, a = tr_get(ta, lane, j), b = tr_get(tb, lane, j);
            if (e < n) put(e, a, b, plain[e] - a - b);
        }
    }
}
__device__ __forceinline__ void put_share(const P6 &out, u64 e, u64 a, u64 b, u64 x3)
{
    out.o[0][e] = a;  out.n[0][e] = b;
    out.o[1][e] = b;  out.n[1][e] = x3;
    out.o[2][e] = x3; out.n[2][e] = a;
}
// the data owner's / query user's role
__global__ __launch_bounds__(256) void k_share(const u32 *keys, u32 op, const u64 *plain, u64 n, P6 out)
{
    __shared__ u64 s_tr[4][2][GT_TR_WORDS];
    const u32 wave = threadIdx.x / GT_LANES;
    share_tiles(keys, GT_KEY_OWNER, op, plain, n, s_tr[wave][0], s_tr[wave][1], [&](u64 e, u64 a, u64 b, u64 x3) { put_share(out, e, a, b, x3); });
}

// The six sharings that the scorer of the heuristic by reconstruction hands back, one launch:
// blockIdx.y = which (operation op + which), under the dealer's key; `off` the first element of
// `out`.  The fourth, the children's node type, goes to both children of a node.  (Six launches and a
// copy before: 34 us a level.)
struct ShareBackArgs { const u32 *keys; u32 op; const u64 *plain[6]; u64 n[6], off[6]; P6 out[6]; };
__global__ __launch_bounds__(256) void k_share_back(ShareBackArgs a)
{
    __shared__ u64 s_tr[4][2][GT_TR_WORDS];
    const u32 wave = threadIdx.x / GT_LANES, q = blockIdx.y;
    const P6 &out = a.out[q];
    const u64 off = a.off[q];
    share_tiles(a.keys, GT_KEY_DEALER, a.op + q, a.plain[q], a.n[q], s_tr[wave][0], s_tr[wave][1], [&](u64 e, u64 x, u64 y, u64 z) {
        if (q == 3) { put_share(out, 2 * (off + e) + 1, x, y, z); put_share(out, 2 * (off + e) + 2, x, y, z); }
        else put_share(out, off + e, x, y, z);
    });
}

// Rec^A: party 0 adds its two components and the one it receives from party 2.
__global__ __launch_bounds__(256) void k_reconstruct(P6 in, u64 n, u64 *plain)
{
    for (u64 e = (u64)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (u64)gridDim.x * blockDim.x)
        plain[e] = in.o[0][e] + in.n[0][e] + in.o[2][e];
}

// local copies of shares, up to three in a launch (blockIdx.y): dst[doff + e] = src[soff + e]
struct CopyArgs { P6 dst[3], src[3]; u64 doff[3], soff[3], n[3]; };
__global__ __launch_bounds__(256) void k_copy(CopyArgs a)
{
    const u32 q = blockIdx.y;
    const P6 &dst = a.dst[q], &src = a.src[q];
    const u64 doff = a.doff[q], soff = a.soff[q];
    for (u64 e = (u64)blockIdx.x * blockDim.x + threadIdx.x; e < a.n[q]; e += (u64)gridDim.x * blockDim.x)
        for (int j = 0; j < 3; j++) {
            dst.o[j][doff + e] = src.o[j][soff + e];
            dst.n[j][doff + e] = src.n[j][soff + e];
        }
}

// dst[k][i] (row stride N8) = src[i][k] (row stride w): sample-contiguous layout.
// 32 x 32 tiles through LDS so that both the reads and the writes are contiguous;
// blockIdx.z selects one of the three components (the own planes).
__global__ __launch_bounds__(256) void k_transpose(P6 dst, P6 src, u32 w, u64 N, u64 N8)
{
    __shared__ u64 tile[32][33];
    const int pl = blockIdx.z, tx = threadIdx.x & 31, ty = threadIdx.x >> 5;       // 32 x 8 threads
    const u64 *in = src.o[pl];
    u64 *out = dst.o[pl];
    const u64 ntx = (w + 31) / 32, nty = (N + 31) / 32;
    for (u64 t = blockIdx.x; t < ntx * nty; t += gridDim.x) {
        const u64 k0 = (t % ntx) * 32, i0 = (t / ntx) * 32;
#pragma unroll
        for (int r = 0; r < 4; r++) {
            const u64 i = i0 + ty + 8 * r, k = k0 + tx;
            tile[ty + 8 * r][tx] = (i < N && k < w) ? in[i * w + k] : 0;
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < 4; r++) {
            const u64 k = k0 + ty + 8 * r, i = i0 + tx;
            if (i < N && k < w) out[k * N8 + i] = tile[tx][ty + 8 * r];
        }
        __syncthreads();
    }
}

// eight consecutive words starting at a multiple of 8: vector loads when all eight lie
// inside the array and the address is 16-byte aligned, guarded loads (zero beyond n) otherwise
__device__ __forceinline__ void ld8(const u64 *ptr, u64 i0, u64 n, u64 (&x)[8])
{
    if (i0 + 8 <= n && ((size_t)(ptr + i0) & 15) == 0) {
        const ulonglong2 *q = (const ulonglong2 *)(ptr + i0);
#pragma unroll
        for (int j = 0; j < 4; j++) { const ulonglong2 v = q[j]; x[2 * j] = v.x; x[2 * j + 1] = v.y; }
    } else {
#pragma unroll
        for (int j = 0; j < 8; j++) x[j] = i0 + j < n ? ptr[i0 + j] : 0;
    }
}

// the same for eight words that exist, 16-byte aligned (whole groups of a plane; rows in LDS)
__device__ __forceinline__ void ld8_whole(const u64 *ptr, u64 (&x)[8])
{
    const ulonglong2 *q = (const ulonglong2 *)ptr;
#pragma unroll
    for (int j = 0; j < 4; j++) { const ulonglong2 v = q[j]; x[2 * j] = v.x; x[2 * j + 1] = v.y; }
}

// every element := public constant c
__global__ __launch_bounds__(256) void k_fill_const(P6 dst, u64 off, u64 n, u64 c)
{
    for (u64 e = (u64)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (u64)gridDim.x * blockDim.x)
        for (int j = 0; j < 3; j++) {
            dst.o[j][off + e] = j == 0 ? c : 0;
            dst.n[j][off + e] = j == 2 ? c : 0;
        }
}

// plain words := c
__global__ __launch_bounds__(256) void k_fill_words(u64 *dst, u64 n, u64 c)
{
    for (u64 e = (u64)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (u64)gridDim.x * blockDim.x) dst[e] = c;
}

// The local steps that end a level (k_split runs them beside the node split): 0: this level's statistics and 1: its
// flags kept for export, 2: T takes the split decisions, 3: children inherit the flags, rows of
// width d: Gn[2r] = Gn[2r+1] = gamma[r] (Sec. V-B; ndup = 0 at the last level).
struct KeepArgs { P6 C, Clast, gamma, Glast, SD, T, Gn; u64 nC, nG, nh, base, ndup; u32 d; };
__device__ __forceinline__ void keep_part(const KeepArgs &a, u32 what, u64 first, u64 step)
{
    const u64 n = what == 0 ? a.nC : (what == 1 ? a.nG : (what == 2 ? a.nh : a.ndup));
    const P6 &src = what == 0 ? a.C : (what == 2 ? a.SD : a.gamma), &dst = what == 0 ? a.Clast : (what == 1 ? a.Glast : (what == 2 ? a.T : a.Gn));
    for (u64 e = first; e < n; e += step) {
        const u64 to = what == 2 ? a.base + e : (what == 3 ? e + e / a.d * a.d : e);
#pragma unroll
        for (int j = 0; j < 3; j++) {
            const u64 vo = src.o[j][e], vn = src.n[j][e];
            dst.o[j][to] = vo; dst.n[j][to] = vn;
            if (what == 3) { dst.o[j][to + a.d] = vo; dst.n[j][to + a.d] = vn; }
        }
    }
}

// ---------------------------------------------------------------------------------
// Limb-tiled layout of the two operands of the statistics contraction.  A 64-bit
// ring element is written as eight signed bytes d_s in [-128,127] with
// x = sum_s d_s 256^s (mod 2^64): add 0x80 to every byte position with carries, then
// flip the top bit of every byte.  A matrix M[row][sample] is stored as
// [sample block of 32][limb s][row][32 bytes], so that one lane of a matrix-core
// operand (one row, 16 consecutive samples, one limb) is one 16-byte load and a
// wavefront reads 1 KB contiguous per limb.  Samples beyond N hold zero bytes.
struct LimbMat { unsigned char *base; u64 rows; };      // rows = row stride of a limb plane
#define GT_BIAS 0x8080808080808080ull

__device__ __forceinline__ u64 limb_addr(const LimbMat &m, u64 ib, u32 s, u64 row) { return ((ib * 8 + s) * m.rows + row) * 32; }

// x[0..8) are 8 consecutive samples (first sample i0, a multiple of 8) of one row
// 8 x 8 byte transpose: afterwards byte j of y[s] is what byte s of y[j] was.  Three
// butterfly stages on byte, 16-bit and 32-bit units; the first two are byte permutes of
// register pairs, the last is a renaming of 32-bit halves.  Its own inverse.
__device__ __forceinline__ void transpose8x8(u64 (&y)[8])
{
    u32 lo[8], hi[8];
#pragma unroll
    for (int j = 0; j < 8; j++) { lo[j] = (u32)y[j]; hi[j] = (u32)(y[j] >> 32); }
#pragma unroll
    for (int j = 0; j < 8; j += 2) {
        const u32 al = lo[j], bl = lo[j + 1], ah = hi[j], bh = hi[j + 1];
        lo[j] = __builtin_amdgcn_perm(bl, al, 0x06020400u); lo[j + 1] = __builtin_amdgcn_perm(bl, al, 0x07030501u);
        hi[j] = __builtin_amdgcn_perm(bh, ah, 0x06020400u); hi[j + 1] = __builtin_amdgcn_perm(bh, ah, 0x07030501u);
    }
#pragma unroll
    for (int j = 0; j < 8; j += 4)
#pragma unroll
        for (int q = 0; q < 2; q++) {
            const u32 al = lo[j + q], bl = lo[j + q + 2], ah = hi[j + q], bh = hi[j + q + 2];
            lo[j + q] = __builtin_amdgcn_perm(bl, al, 0x05040100u); lo[j + q + 2] = __builtin_amdgcn_perm(bl, al, 0x07060302u);
            hi[j + q] = __builtin_amdgcn_perm(bh, ah, 0x05040100u); hi[j + q + 2] = __builtin_amdgcn_perm(bh, ah, 0x07060302u);
        }
#pragma unroll
    for (int q = 0; q < 4; q++) {
        y[q] = (u64)lo[q] | ((u64)lo[q + 4] << 32);
        y[q + 4] = (u64)hi[q] | ((u64)hi[q + 4] << 32);
    }
}

__device__ __forceinline__ void store_limbs8(const LimbMat &m, u64 row, u64 i0, const u64 (&x)[8])
{
    u64 y[8];
#pragma unroll
    for (int j = 0; j < 8; j++) y[j] = (x[j] + GT_BIAS) ^ GT_BIAS;
    transpose8x8(y);                                  // byte j of y[s] is limb s of sample j
    const u64 ib = i0 >> 5;
    const u32 off = (u32)i0 & 31;
#pragma unroll
    for (int sl = 0; sl < 8; sl++) *(u64 *)(m.base + limb_addr(m, ib, sl, row) + off) = y[sl];
}

// value of sample i of a row
__device__ __forceinline__ u64 load_limbs1(const LimbMat &m, u64 row, u64 i)
{
    u64 y = 0;
#pragma unroll
    for (int sl = 0; sl < 8; sl++) y |= (u64)m.base[limb_addr(m, i >> 5, sl, row) + (i & 31)] << (8 * sl);
    return (y ^ GT_BIAS) - GT_BIAS;
}

// The operands of the contraction z_p = x_p (y_p + y_{p+1}) + x_{p+1} y_p (the three-term
// product of Sec. II-B with the sum moved to one factor): x is stored once per COMPONENT -
// component j is what party j holds as its own and party j-1 as its next part, the two
// copies are equal by construction, party j's wavefront writes the one that both holders
// read - and y per party as (own+next, own).  L, the leaf one-hot made anew at every level, has
// 2^h rows, B, the columns made at set-up, has d*K + K.  The operand with fewer rows takes the
// role of y (and is written twice), so that the larger one is written and read once per
// component: for 48,842 x 294 columns and 2 classes the contraction reads 0.69 GB per level
// instead of 1.38.  The class totals of the label level always take L as x.
struct LimbSet { LimbMat m[3][2]; };
struct LimbTri { LimbMat m[3]; };

// ---------------------------------------------------------------------------------
// Elementwise product (Sec. II-B), 8 elements per lane, consecutive ones in consecutive lanes.
// MODE 0: z[e] = x[e]*y[e].
// MODE 2 (node split): e = r*CW + col, z = C[e] * (1 - split[r]), written to both
//         children (2r, 2r+1) of the next level.
// The zero-sharing words under key k_j are evaluated by party j's wavefront and also loaded by
// party j-1, the other holder of that key.  Bound: memory.  2^24 products:
// 0.92 ms with lanes on 8 consecutive elements each and both keys' blocks per party, 0.50 ms with the six planes of each factor
// read (12 words, 4.8 TB/s), 0.36 ms with each component of the factors read once, for both of its holders, from the plane of the party whose own
// it is (6 words read, 6 written).  In place is safe: a barrier lies between the loads of a half tile and its stores.
struct MultArgs { KCommon c; P6 x, y, z; u64 n; u32 CW; };   // CW: MODE 2

template <int MODE, bool EARLY = false>
__device__ __forceinline__ void mult_tiles(const MultArgs &a, u32 block, u32 blocks)
{
    const int p = party_of_wave(), lane = threadIdx.x, pn = p == 2 ? 0 : p + 1;
    __shared__ u64 s_wire[GT_LWIRE_WORDS];
    __shared__ u64 s_tr[3][GT_TR_WORDS];
    __shared__ u64 s_cnt[6];
    Wire W; W.init(s_wire, s_cnt);
    const Key own = load_key(a.c.keys, p);
    const u64 *xo = own_of(a.x, p), *xn = nxt_of(a.x, p), *yo = own_of(a.y, p), *yn = nxt_of(a.y, p);
    u64 *zo = own_of(a.z, p), *zn = nxt_of(a.z, p);
    const Sh one = pub(p, 1);
    const bool narrow = a.n <= 0xffffffffu;            // 32-bit division: a tenth of the instructions of the 64-bit one
    for (u64 tile = block, nt = (a.n + 511) / 512; tile < nt; tile += blocks) {
        u64 w[8];
        Sh px[8], py[8];
        if (EARLY) {                                   // in flight during the block function
#pragma unroll
            for (int j = 0; j < 8; j++) {
                const u64 e = tile * 512 + j * GT_LANES + lane, el = e < a.n ? e : a.n - 1;
                const u64 r = narrow ? (u64)((u32)el / a.CW) : el / a.CW;
                px[j].o = xo[el]; px[j].n = xn[el]; py[j].o = yo[r]; py[j].n = yn[r];
            }
        }
        chacha8(own, tile * GT_LANES + lane, a.c.op, 0, w);
        tr_put(s_tr[p], lane, w);
        __syncthreads();
#pragma unroll
        for (int h = 0; h < 2; h++) {
            u64 snd[4], rcv[4], at[4];
            u32 live = 0;
#pragma unroll
            for (int i = 0; i < 4; i++) {
                const int j = 4 * h + i;
                const u64 e = tile * 512 + j * GT_LANES + lane;
                const u64 alpha = tr_get(s_tr[p], lane, j) - tr_get(s_tr[pn], lane, j);
                Sh x = { 0, 0 }, y = { 0, 0 };
                at[i] = e;
                if (e < a.n) {
                    live++;
                    if (MODE == 0) { x.o = xo[e]; x.n = xn[e]; y.o = yo[e]; y.n = yn[e]; }
                    if (MODE == 2) {
                        const u64 r = narrow ? (u64)((u32)e / a.CW) : e / a.CW;
                        if (EARLY) { x = px[j]; y = one - py[j]; }
                        else { x.o = xo[e]; x.n = xn[e]; y.o = one.o - yo[r]; y.n = one.n - yn[r]; }
                        at[i] = e + r * a.CW;          // element (2r, col) of the next level
                    }
                }
                snd[i] = prod3(x, y) + alpha;
            }
            W.reshare<4>(snd, rcv, 64u * live);
#pragma unroll
            for (int i = 0; i < 4; i++) {
                if (tile * 512 + (4 * h + i) * GT_LANES + lane < a.n) {
                    zo[at[i]] = snd[i]; zn[at[i]] = rcv[i];
                    if (MODE == 2) { zo[at[i] + a.CW] = snd[i]; zn[at[i] + a.CW] = rcv[i]; }
                }
            }
        }
        __syncthreads();                               // the words in LDS are overwritten next
    }
    W.flush(a.c.wire);
}
__global__ __launch_bounds__(192) void k_mult(MultArgs a) { mult_tiles<0>(a, blockIdx.x, gridDim.x); }
// End of a level in one launch: the first mblk workgroups the children's statistics, the others (in fours) the local copies.
// (Two launches, each a few microseconds at small levels: training of 267 x 22, depth 4.)  EARLY: 145 registers, 3 wavefronts per SIMD (102, 4): see split_early
template <bool EARLY>
__global__ __launch_bounds__(192) void k_split(MultArgs m, KeepArgs k, u32 mblk)
{
    if (blockIdx.x < mblk) mult_tiles<2, EARLY>(m, blockIdx.x, mblk);
    else {
        const u32 b = blockIdx.x - mblk, nb = (gridDim.x - mblk) / 4;
        keep_part(k, b & 3, (u64)(b >> 2) * 192 + threadIdx.y * GT_LANES + threadIdx.x, (u64)nb * 192);
    }
}

// What a training computes once, one launch: the sample-contiguous copies XT[k][i] and YT[c][i] of the data (a plane per component), the one-time
// products of the learning protocol (Sec. V-B) and the class columns, as limb tiles.  Product column col = k*K + c, element
// e = col*N8 + i, z = X[i][k] * Y[i][c] for i < N, as rows 0 .. d*K - 1 of C (COMPS: the columns once per component) or of B (own + next
// component into B.m[p][0], own into B.m[p][1]); class column c as row c of Yl (both forms) and, with COMPS, row d*K + c of C.
// A workgroup takes 32 samples (a sample block) x tk features: rows of X and Y through LDS, where its four wavefronts read them: a
// wavefront is the three parties on the block x 5 adjacent columns per step, so that the 32-byte pieces that a party's lanes write per limb
// lie side by side.
// Bound: memory (1.5 GB of X read, 1.5 of XT and 6.1 of tiles written at 10^6 x 64, 4 classes, in 2.44 ms: 3.7 TB/s), the vector ALU close
// behind (the tiles' stores alone 1.6 ms, all but these 1.6).  Three workgroups per compute unit, each grid-stride over its items: a workgroup for every
// item, whose message counters then queue at 64 lines, took 3.4 ms, with the rows' loads one after the other 3.0.  Rows of eight words from global memory by
// the lanes that use them: 3.4 ms, each load instruction touches as many lines as it has lanes.  One wavefront per party with a barrier per message, after a
// transposition, before class tiles of their own: 2.49 + 0.73 + 0.31 ms; 48,842 x 294, 2 classes 369 + 150 + 20 us, now 357; 19,997 x 101, 3
// classes 118 + 25 + 10, now 74; 267 x 22 15 + 5 + 5, now 8.  The 168 registers of three wavefronts per SIMD spill 9 and, without COMPS, 21 (11 and 23 with 16 classes).
struct XyArgs { KCommon c; P6 X, Y, XT, YT; LimbSet B, Yl; LimbTri C; u64 N, N8; u32 d, K, tk; };
#define GT_XY_ROW 34                                   // words of a row in LDS: 32 samples, 16 bytes further on in the banks
template <bool COMPS, int KMAX>
__global__ __launch_bounds__(256, 3) void k_xy(XyArgs a)
{
    __shared__ uint4 s_msg[4][GT_WMSG_QUADS];
    __shared__ u64 s_cnt[4][6];
    __shared__ __align__(16) u64 s_x[3 * GT_XY_FEAT * GT_XY_ROW], s_y[3 * KMAX * GT_XY_ROW];
    const u32 wave = __builtin_amdgcn_readfirstlane(threadIdx.x / GT_LANES), tid = threadIdx.x;
    WWire W; W.init(s_msg[wave], s_cnt[wave]);
    const int p = W.p;
    const Key own = load_lane_key(a.c.keys, p);
    const u64 ngrp = a.N8 / 8, nt = (ngrp + 3) / 4;
    const u32 t = W.t < 4 * GT_XY_COLS ? W.t : 4 * GT_XY_COLS - 1, ro = t / 4, gi = t % 4;
    const LimbMat zo = COMPS ? (p == 0 ? a.C.m[0] : (p == 1 ? a.C.m[1] : a.C.m[2])) : (p == 0 ? a.B.m[0][1] : (p == 1 ? a.B.m[1][1] : a.B.m[2][1]));
    const LimbMat zs = p == 0 ? a.B.m[0][0] : (p == 1 ? a.B.m[1][0] : a.B.m[2][0]);
    const LimbMat lo = p == 0 ? a.Yl.m[0][1] : (p == 1 ? a.Yl.m[1][1] : a.Yl.m[2][1]), ls = p == 0 ? a.Yl.m[0][0] : (p == 1 ? a.Yl.m[1][0] : a.Yl.m[2][0]);
    const u32 nkt = (a.d + a.tk - 1) / a.tk;
    for (u64 item = blockIdx.x; item < nt * nkt; item += gridDim.x) {
        const u64 tile = item / nkt, is = tile * 32;
        const u32 k0 = (u32)(item % nkt) * a.tk, nk = k0 + a.tk < a.d ? a.tk : a.d - k0;
        // rows of X and Y: consecutive words in consecutive threads, all loads before the first wait; samples beyond N are zero
        {
            constexpr int NY = (32 * KMAX + 255) / 256;
            const u32 k = tid % GT_XY_FEAT, i = tid / GT_XY_FEAT;
            u64 x[4][3], y[NY][3];
#pragma unroll
            for (int r = 0; r < 4; r++) {
                const u64 row = is + i + 8 * r;
                const u64 at = (row < a.N ? row : a.N - 1) * a.d + k0 + (k < nk ? k : 0);
#pragma unroll
                for (int j = 0; j < 3; j++) x[r][j] = a.X.o[j][at];
            }
#pragma unroll
            for (int q = 0; q < NY; q++) {
                const u64 at = is * a.K + tid + 256 * q, n = a.N * a.K;
#pragma unroll
                for (int j = 0; j < 3; j++) y[q][j] = a.Y.o[j][at < n ? at : n - 1];
            }
#pragma unroll
            for (int r = 0; r < 4; r++)
#pragma unroll
                for (int j = 0; j < 3; j++) s_x[(j * GT_XY_FEAT + k) * GT_XY_ROW + i + 8 * r] = is + i + 8 * r < a.N ? x[r][j] : 0;
#pragma unroll
            for (int q = 0; q < NY; q++) {
                const u32 e = tid + 256 * q, s = e / a.K, c = e - s * a.K;
                if (e < 32 * a.K) {
#pragma unroll
                    for (int j = 0; j < 3; j++) s_y[(j * KMAX + c) * GT_XY_ROW + s] = is + s < a.N ? y[q][j] : 0;
                }
            }
        }
        __syncthreads();
        for (u32 e = tid; e < 3 * 16 * nk; e += 256) {          // two samples each
            const u32 i = e % 16 * 2, r = e / 16, j = r / nk, k = r - j * nk;
            if (is + i < a.N8) *(ulonglong2 *)(a.XT.o[j] + (k0 + k) * a.N8 + is + i) = *(const ulonglong2 *)&s_x[(j * GT_XY_FEAT + k) * GT_XY_ROW + i];
        }
        const u64 g = tile * 4 + gi, grp = g < ngrp ? g : ngrp - 1, i0 = grp * 8;
        const u32 off = (u32)(i0 - is);                        // the lane's first sample in the block
        const bool actg = W.t < 4 * GT_XY_COLS && g < ngrp;    // the same in lane 63 as in lane 62
        const auto row8 = [&](const u64 *row, u64 (&x)[8]) { ld8_whole(row + off, x); };
        if (k0 == 0) {
            for (u32 e = tid; e < 3 * 16 * a.K; e += 256) {
                const u32 i = e % 16 * 2, r = e / 16, j = r / a.K, c = r - j * a.K;
                if (is + i < a.N8) *(ulonglong2 *)(a.YT.o[j] + c * a.N8 + is + i) = *(const ulonglong2 *)&s_y[(j * KMAX + c) * GT_XY_ROW + i];
            }
            for (u32 c0 = wave * GT_XY_COLS; c0 < a.K; c0 += 4 * GT_XY_COLS) {
                const u32 c = c0 + ro < a.K ? c0 + ro : a.K - 1;
                u64 yo[8], yn[8];
                row8(s_y + (p * KMAX + c) * GT_XY_ROW, yo); row8(s_y + (W.pn * KMAX + c) * GT_XY_ROW, yn);
                store_limbs8(lo, c, i0, yo);
                if (COMPS) store_limbs8(zo, (u64)a.d * a.K + c, i0, yo);
#pragma unroll
                for (int s = 0; s < 8; s++) yn[s] += yo[s];
                store_limbs8(ls, c, i0, yn);
            }
        }
        const bool tail = __ballot(i0 + 8 > a.N) != 0;         // uniform: a branch instead of 32 selections per step
        const u32 kend = (k0 + nk) * a.K;
        // lanes without an element of their own repeat another's, so that no store needs a branch
        for (u32 kb = k0 * a.K + wave * GT_XY_COLS; kb < kend; kb += 4 * GT_XY_COLS) {
            const u32 col = kb + ro < kend ? kb + ro : kend - 1, k = col / a.K, c = col - k * a.K;
            u64 ao[8], an[8], snd[8], rcv[8];
            chacha8<PRF_PAIR_LOOP>(own, (u64)col * ngrp + grp, a.c.op, 0, ao);
            W.pass64<8>(ao, an, W.nx);                         // the words under the next key, from the other holder of that key
            const u64 *xr = s_x + (p * GT_XY_FEAT + k - k0) * GT_XY_ROW + off, *xq = s_x + (W.pn * GT_XY_FEAT + k - k0) * GT_XY_ROW + off;
            const u64 *yr = s_y + (p * KMAX + c) * GT_XY_ROW + off, *yq = s_y + (W.pn * KMAX + c) * GT_XY_ROW + off;
#pragma unroll
            for (int s = 0; s < 8; s += 2) {
                const ulonglong2 xo = *(const ulonglong2 *)(xr + s), xn = *(const ulonglong2 *)(xq + s), yo = *(const ulonglong2 *)(yr + s), yn = *(const ulonglong2 *)(yq + s);
                snd[s] = prod3(Sh{ xo.x, xn.x }, Sh{ yo.x, yn.x }) + (ao[s] - an[s]);
                snd[s + 1] = prod3(Sh{ xo.y, xn.y }, Sh{ yo.y, yn.y }) + (ao[s + 1] - an[s + 1]);
            }
            W.reshare64<8>(snd, rcv);
            W.nresh += actg && kb + ro < kend ? 64u * live8(i0, a.N) : 0u;
            if (tail) {
#pragma unroll
                for (int s = 0; s < 8; s++) if (i0 + s >= a.N) { snd[s] = 0; rcv[s] = 0; }
            }
            store_limbs8(zo, col, i0, snd);
            if (!COMPS) {
#pragma unroll
                for (int s = 0; s < 8; s++) rcv[s] += snd[s];
                store_limbs8(zs, col, i0, rcv);
            }
        }
        W.drain();
        __syncthreads();                                       // the rows in LDS are overwritten next
    }
    W.flush(a.c.wire);
}

// what a training starts from, one launch (blockIdx.y): M, T, C := 0; F := 0, the root a leaf (1); gamma of the
// root := 1
struct StartArgs { P6 M, T, F, C, gamma; u64 N, nodes, nC, d; };
__global__ __launch_bounds__(256) void k_start(StartArgs a)
{
    const u32 what = blockIdx.y;
    const u64 n = what == 0 ? a.N : (what == 3 ? a.nC : (what == 4 ? a.d : a.nodes));
    const P6 &dst = what == 0 ? a.M : (what == 1 ? a.T : (what == 2 ? a.F : (what == 3 ? a.C : a.gamma)));
    for (u64 e = (u64)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (u64)gridDim.x * blockDim.x) {
        const u64 c = what == 4 || (what == 2 && e == 0) ? 1 : 0;
#pragma unroll
        for (int j = 0; j < 3; j++) { dst.o[j][e] = j == 0 ? c : 0; dst.n[j][e] = j == 2 ? c : 0; }
    }
}

// per-sample leaf one-hot back to 64-bit words for export: out[r*N8 + i]
__global__ __launch_bounds__(256) void k_l_export(LimbTri L, P6 out, u64 nh, u64 N, u64 N8)
{
    const u64 total = nh * N8;
    for (u64 t = (u64)blockIdx.x * blockDim.x + threadIdx.x; t < total; t += (u64)gridDim.x * blockDim.x) {
        const u64 r = t / N8, i = t % N8;
        for (int p = 0; p < 3; p++) {
            u64 own = 0, nxt = 0;
            if (i < N) { own = load_limbs1(L.m[p], r, i); nxt = load_limbs1(L.m[p == 2 ? 0 : p + 1], r, i); }
            out.o[p][t] = own; out.n[p][t] = nxt;
        }
    }
}

// ---------------------------------------------------------------------------------
// Equality grid (first lines of the array-access protocol, Sec. V-A; per-sample leaf
// flags of the learning protocol, Sec. V-B).  Rows are samples i < N, columns k < w;
// element (k, i) has index k*N8 + i.  A lane owns 8 consecutive samples and walks
// over the columns, so that one PRF block yields the mask words of its 8 elements
// and the inner products of the array access accumulate in registers.
//   E[k][i] = [u[i] - base == k]  (and g[k] if HAS_G)  -> arithmetic sharing, then
//   GM_STORE : E written as limb tiles, the left operand of the statistics contraction
//   GM_COMMON: z[i] = sum_k E[k][i] * W1[w1off+k]   (NDOT = 2: also W2 -> out2)
//   GM_ROWS  : z[i] = sum_k E[k][i] * XT[k*N8+i]
//   epilogue 0: out[i] = z;  1: out[i] = 2*prev[i] + z + 1  (index update of the
//   partition and inference protocols).
struct GridArgs {
    KCommon c;
    P6 u; u64 base; u32 w; u64 N, N8;
    P6 g, out, out2, W1, W2, XT, prev;
    u64 w1off, w2off;
    int epi;
    LimbTri L, S;   // GM_STORE: limb tiles of the components, row = column k; S (sums): party p's own+next
    int sums;
    u32 nkc, kchunk;// column ranges per tile and their length
    u32 gpt, rps;   // groups of 8 samples per tile, adjacent columns per step (gpt * rps <= 21)
    u64 *dacc;      // [2][3][N8] partial inner products when nkc > 1
    int ndot;
};

// Eight equality tests of one lane (one column, eight rows) in the wavefront model.
//
// The AND rounds work on packed fields from the second round on, so that one word operation
// serves several tests; the two halves of the fields are separated before the AND, so that
// its result is the next message as it stands: fields of 16 bits (two tests per dword), 8
// bits (four), then nibbles, two bits in a nibble, one bit in a nibble (eight tests in one
// dword: test s < 4 in nibble 2s, test s >= 4 in nibble 2(s-4)+1).  Mask words (own xor next
// key): bits 0-31 round 0, 32-47 round 1, 48-55 round 2, 56-59 round 3, 60-61 round 4, 62
// round 5, 63 an AND that follows.
//
// Offline and pairwise-key material is evaluated once and handed out through LDS: the daBits
// of the eight tests come from three dealer blocks (stream 4, blocks 3g..3g+2 of the group
// g = e/8; test j in slot j%3 of block 3g + j/3), one in the lane of each party (the dealer is a
// role of its own: a block yields the components of all three parties, each party then loads
// its two); the mask words under key k_j are evaluated by party j's lane and also loaded by
// party j-1, the other holder of k_j.
#define GT_EQ_NIB 0x11111111u
__host__ __device__ constexpr int eq_pos(int s) { return s < 4 ? 8 * s : 8 * (s - 4) + 4; }     // bit of test s after the rounds
// Rows of the daBit components in LDS, a word per lane of a party: component c of test s at eq_row(c, s).  The three tests that the parties
// deal together lie side by side, and a component's rows are 21 words on from the one before modulo 32, so that neither the dealing
// lanes' stores nor the parties' loads, each of another component, meet in a bank.
#define GT_EQ_COMP (9 * GT_TP + 24)              // 9 tests, one unused; 213 = 21 modulo 32
#define GT_EQ_ROWS (2 * GT_EQ_COMP + 9 * GT_TP)
__host__ __device__ constexpr int eq_row(int c, int s) { return c * GT_EQ_COMP + (s % 3 * 3 + s / 3) * GT_TP; }

struct EqWave {
    WWire W;
    Key own, dlr;
    u64 *rows;                   // GT_EQ_ROWS words of the wavefront
    u32 M0, M2;                  // all ones in the lanes of party 0 / party 2, the holders of component 0
    u32 sh0, sh1, sh2, k2;       // positions of the three tests whose daBits this lane deals; k2: the third exists

    __device__ __forceinline__ void init(const u32 *keys, uint4 *region, u64 *s_rows, u64 *s_cnt)
    {
        W.init(region, s_cnt);
        own = load_lane_key(keys, W.p); dlr = load_key(keys, GT_KEY_DEALER);
        rows = s_rows;
        M0 = W.p == 0 ? ~0u : 0u; M2 = W.p == 2 ? ~0u : 0u;
        sh0 = W.p == 0 ? eq_pos(0) : (W.p == 1 ? eq_pos(3) : eq_pos(6));
        sh1 = W.p == 0 ? eq_pos(1) : (W.p == 1 ? eq_pos(4) : eq_pos(7));
        sh2 = W.p == 0 ? eq_pos(2) : (W.p == 1 ? eq_pos(5) : 0);
        k2 = W.p == 2 ? 0u : 7u;
    }
    // daBit component c of this lane's test s
    __device__ __forceinline__ u64 &row(int c, int s) { return rows[c * GT_EQ_COMP + eq_row(0, s) + W.t]; }

    // The daBits of the eight tests of block index g of operation op: this lane's block, components to the rows of `r` (row(0, 0)
    // of a row area: COMP words from a component to the next, STEP from the lane's test to its next, PARTY from a party's first test to the
    // next party's); returns the Boolean components of its three tests, in their positions.
    template <int ISSUE, int COMP = GT_EQ_COMP, int STEP = 3 * GT_TP, int PARTY = GT_TP>
    __device__ __forceinline__ u32 deal_bits(u32 op, u64 g, u64 *r)
    {
        u64 D[8];
        chacha8<ISSUE>(dlr, 3 * g + (u32)W.p, op, 4, D);
        wave_sync();
        const u32 x = (u32)D[6] & 0x1ffu;
        r += W.p * PARTY;
#pragma unroll
        for (int q = 0; q < 3; q++) {
            u64 *rq = r + q * STEP;
            rq[0] = D[2 * q]; rq[COMP] = D[2 * q + 1];
            rq[2 * COMP] = (u64)((x >> (3 * q)) & 1) - D[2 * q] - D[2 * q + 1];
        }
        // per test three Boolean components in a nibble: bits 1, 2 of its field and beta xor both
        const u32 z = ((x >> 1) & 0xdbu) | ((xor3l(x, x >> 1, x >> 2) & 0x49u) << 2);
        return ((z & 7) << sh0) | (((z >> 3) & 7) << sh1) | (((z >> 6) & k2) << sh2);
    }

    // [c - base - k == 0] (and the shared bit g) for the eight rows of block index g of operation
    // op.  state(h, cd, ro, rn) fetches what rows h .. h + 3 are tested with: cd = c - base - k (public), ro and rn the Boolean
    // components of r.  Returns the opened f = result xor beta, test s in bit eq_pos(s); beta's arithmetic components are in row(.,s).
    // early(): the loads of what the tests' results meet, issued after the PRF blocks (their registers
    // are free again) and in flight during the rounds.
    template <bool HAS_G, int ISSUE, class S, class F>
    __device__ __forceinline__ u32 tests(u32 op, u64 g, S state, u32 go, u32 gn, u32 nl, F early)
    {
        u32 b1[1] = { deal_bits<ISSUE>(op, g, &row(0, 0)) }, b2[1];
        W.pass<1>(b1, b2, W.nx);
        const u32 bw = b1[0] | b2[0] | W.buf[W.pv].x;
        u64 A[8];
        chacha8<ISSUE>(own, g, op, 1, A);
        return rounds<HAS_G>(A, bw, state, go, gn, nl, early);
    }

    // The rounds of the eight tests: A the mask words under the party's own key (those under the other come from the next party,
    // four tests at a time: fewer registers, half the message region), bw the Boolean components of the daBits.
    template <bool HAS_G, class S, class F>
    __device__ __forceinline__ u32 rounds(const u64 (&A)[8], u32 bw, S state, u32 go, u32 gn, u32 nl, F early)
    {
        u32 Ah[8], xo[8], xn[8];
        // round 0, width 32: the high word onto the low word
#pragma unroll
        for (int h = 0; h < 8; h += 4) {
            const u64 A4[4] = { A[h], A[h + 1], A[h + 2], A[h + 3] };
            u64 An[4];
            W.pass64<4>(A4, An, W.nx);
            u64 cd[4], ro[4], rn[4];
            state(h, cd, ro, rn);
#pragma unroll
            for (int j = 0; j < 4; j++) {
                const int s = h + j;
                const u32 dl = (u32)cd[j], dh = (u32)(cd[j] >> 32);
                // t = rho with the complement of cd xored into component 0
                const u32 tol = logic3<0xd2>((u32)ro[j], dl, M0), toh = logic3<0xd2>((u32)(ro[j] >> 32), dh, M0);
                const u32 tnl = logic3<0xd2>((u32)rn[j], dl, M2), tnh = logic3<0xd2>((u32)(rn[j] >> 32), dh, M2);
                xo[s] = xor3l(and3l(tol, tnl, toh, tnh), (u32)A[s], (u32)An[j]);
                Ah[s] = (u32)(A[s] >> 32) ^ (u32)(An[j] >> 32);
            }
        }
        early();
        W.reshare<8>(xo, xn);
        u32 Po[4], Pn[4], H[4];
#pragma unroll
        for (int j = 0; j < 4; j++) {                  // round 1, width 16
            const u32 al = __builtin_amdgcn_perm(xo[2 * j + 1], xo[2 * j], 0x05040100u), ah = __builtin_amdgcn_perm(xo[2 * j + 1], xo[2 * j], 0x07060302u);
            const u32 bl = __builtin_amdgcn_perm(xn[2 * j + 1], xn[2 * j], 0x05040100u), bh = __builtin_amdgcn_perm(xn[2 * j + 1], xn[2 * j], 0x07060302u);
            Po[j] = and3l(al, bl, ah, bh) ^ __builtin_amdgcn_perm(Ah[2 * j + 1], Ah[2 * j], 0x05040100u);
            H[j] = __builtin_amdgcn_perm(Ah[2 * j + 1], Ah[2 * j], 0x07060302u);
        }
        W.reshare<4>(Po, Pn);
        u32 Qo[2], Qn[2], B3[2];
#pragma unroll
        for (int j = 0; j < 2; j++) {                  // round 2, width 8
            const u32 al = __builtin_amdgcn_perm(Po[2 * j + 1], Po[2 * j], 0x06040200u), ah = __builtin_amdgcn_perm(Po[2 * j + 1], Po[2 * j], 0x07050301u);
            const u32 bl = __builtin_amdgcn_perm(Pn[2 * j + 1], Pn[2 * j], 0x06040200u), bh = __builtin_amdgcn_perm(Pn[2 * j + 1], Pn[2 * j], 0x07050301u);
            Qo[j] = and3l(al, bl, ah, bh) ^ __builtin_amdgcn_perm(H[2 * j + 1], H[2 * j], 0x06040200u);
            B3[j] = __builtin_amdgcn_perm(H[2 * j + 1], H[2 * j], 0x07050301u);
        }
        W.reshare<2>(Qo, Qn);
        const u32 LN = 0x0f0f0f0fu;
        // per byte the low nibble of x, the high nibble of y
#define GT_NIBS(x, y) logic3<0xac>(LN, y, x)
        u32 Ro[1], Rn[1];                              // round 3, width 4
        Ro[0] = and3l(GT_NIBS(Qo[0], Qo[1] << 4), GT_NIBS(Qn[0], Qn[1] << 4), GT_NIBS(Qo[0] >> 4, Qo[1]), GT_NIBS(Qn[0] >> 4, Qn[1]))
                ^ GT_NIBS(B3[0], B3[1] << 4);
        W.reshare<1>(Ro, Rn);
        const u32 Hm = GT_NIBS(B3[0] >> 4, B3[1]);     // bits 60-63 of the mask words, one nibble per test
#undef GT_NIBS
        u32 So[1], Sn[1];                              // round 4, width 2
        So[0] = logic3<0x60>(0x33333333u, and3l(Ro[0], Rn[0], Ro[0] >> 2, Rn[0] >> 2), Hm);
        W.reshare<1>(So, Sn);
        u32 To[1], Tn[1];                              // round 5, width 1
        To[0] = (and3l(So[0], Sn[0], So[0] >> 1, Sn[0] >> 1) ^ (Hm >> 2)) & GT_EQ_NIB;
        W.reshare<1>(To, Tn);
        if (HAS_G) {                                   // and with the column's shared bit (go, gn: that bit in every position)
            To[0] = (and3l(To[0], Tn[0], go, gn) ^ (Hm >> 3)) & GT_EQ_NIB;
            W.reshare<1>(To, Tn);
        }
        // bit -> arithmetic: open s xor beta
        u32 fo[1] = { (To[0] ^ (bw >> W.p)) & GT_EQ_NIB }, fr[1];
        W.pass<1>(fo, fr, W.pv);
        W.nopen += nl; W.nresh += (HAS_G ? 64u : 63u) * nl;
        return xor3l(fo[0], Tn[0] ^ (bw >> W.pn), fr[0]);
    }

    // Row part of a grid: the edaBits of the lane's eight rows (dealer blocks i0..i0+7 of stream
    // 0, split over the lanes of the three parties), the masked values and their one opening.
    // u: the rows' values (in: own, next).  cpub = u + r, rho: Boolean components of r.
    template <int ISSUE>
    __device__ __forceinline__ void open_rows(u32 op, u64 i0, const u64 (&uo)[8], const u64 (&un)[8], u64 (&cpub)[8],
                                              u64 (&rho_o)[8], u64 (&rho_n)[8], u32 bits)
    {
        u64 keep[3][3], snd[8], mn[8], rcv[8];
#pragma unroll
        for (int h = 0; h < 2; h++) {                  // arithmetic components, then the Boolean ones, through the same rows
#pragma unroll
            for (int q = 0; q < 3; q++) {
                const int s = 3 * W.p + q;             // s = 8 (party 2): the unused row
                u64 *r = rows + (3 * q + W.p) * GT_TP + W.t;           // row(0, s)
                if (h == 0) {
                    u64 D[8];
                    chacha8<ISSUE>(dlr, i0 + (u32)s, op, 0, D);
                    wave_sync();
                    r[0] = D[1]; r[GT_EQ_COMP] = D[2]; r[2 * GT_EQ_COMP] = D[0] - D[1] - D[2];
                    keep[q][0] = D[3]; keep[q][1] = D[4]; keep[q][2] = D[0] ^ D[3] ^ D[4];
                } else { r[0] = keep[q][0]; r[GT_EQ_COMP] = keep[q][1]; r[2 * GT_EQ_COMP] = keep[q][2]; }
            }
            wave_sync();
#pragma unroll
            for (int s = 0; s < 8; s++) {
                if (h == 0) { snd[s] = uo[s] + row(W.p, s); mn[s] = un[s] + row(W.pn, s); }
                else { rho_o[s] = row(W.p, s); rho_n[s] = row(W.pn, s); }
            }
            wave_sync();
        }
        W.open64<8>(snd, rcv);
        W.nopen += bits;
#pragma unroll
        for (int s = 0; s < 8; s++) cpub[s] = snd[s] + mn[s] + rcv[s];
    }
};

// the columns' part of E: f ? 1 - b : b for one component, m = all ones where f is set, k1 = that
// party's component of the public 1, plus 1 (f ? one - b : b = (b xor m) + (m & (one + 1)))
__device__ __forceinline__ u64 eq_select(u64 b, u32 m, u32 k1) { return (b ^ ((u64)m | ((u64)m << 32))) + (u64)(m & k1); }

// Equality grid (first lines of the array-access protocol, Sec. V-A; per-sample leaf flags of
// the learning protocol, Sec. V-B): see GridArgs for the modes.
// Bound: vector ALU.  A step (168 tests) executes 1,070 vector instructions, 700 of them PRF (two thirds of these can pair, see chacha8), and
// with two wavefronts per SIMD 31 % of a wavefront's time is waiting: 19 for LDS (messages, daBits), 12 for the issue.  WAVES 3: a third one
// fills that.  Its 168 registers hold the keys, the sums and a step's words but for 19 (leaf one-hot) and 22 (80 and 92 bytes a lane in scratch, which
// shows in the bytes written); the rows' public values and Boolean components are read from LDS in every step (12.5 KB a wavefront).  WAVES 2: they stay in registers (none spill), for launches that do not fill three,
// and for the samples' own values (GM_ROWS), which are fetched a step ahead and take the registers of the third.  A step
// takes 3,750 cycles of a SIMD with two and 3,400 with three: 1,000,000 x 64 583 and 528 us (x 512 11.4 and 12.9 * 10^10 tests/s),
// array access 200,003 x 100 211 and 195 us, leaf one-hot of 48,842 x (128 + 256 nodes) 307 and 225; but own rows 100,000 x 100 135 and 145,
// 48,842 x 64, which fills two per SIMD, 46.5 and 50.2.  Which: column_ranges.  One wavefront per workgroup.
// Earlier: one party per wavefront and ten workgroup barriers per step, then without paired additions, then with them: array access
// 0.40, 0.27, 0.21 ms; 10^6 samples x (64 + 128 nodes) 3.45, 2.67, 2.14 (now 1.95), own rows 2 x 64 columns 2.35, 1.77, 1.5 ms,
// leaf grid of 128 + 256 nodes 6.3, 6.2, 5.9 (now 5.6) ms.
template <int MODE, bool HAS_G, int NDOT, int ISSUE, int WAVES>
__global__ __launch_bounds__(64, WAVES) void k_eqgrid(GridArgs a)
{
    __shared__ uint4 s_msg[GT_WMSG_QUADS];
    __shared__ u64 s_rows[GT_EQ_ROWS];
    __shared__ u64 s_cnt[6];
    static_assert(WAVES == 2 || (MODE != GM_ROWS && NDOT == 1), "own rows and two sums take two wavefronts per SIMD");
    constexpr bool IN_LDS = WAVES > 2;                 // the rows' opened values and Boolean components
    __shared__ ulonglong2 s_rho[IN_LDS ? 4 * GT_LANES : 1], s_open[IN_LDS ? 4 * GT_TP : 1];
    EqWave E;
    E.init(a.c.keys, s_msg, s_rows, s_cnt);
    WWire &W = E.W;
    const int p = W.p;
    const u32 op = a.c.op;
    const u64 ngrp = a.N8 / 8;
    const Sh one = pub(p, 1);
    const u32 k1o = (u32)one.o + 1, k1n = (u32)one.n + 1;
    // work item = (tile of gpt groups of 8 samples, range of columns); with more than one column
    // range per tile the inner products are completed by atomic adds (exact in the ring) and
    // the reshare runs in k_dot_fin.  A step covers rps adjacent columns of the tile.
    const u32 gpt = a.gpt, ro = W.t / gpt, gi = W.t - ro * gpt;
    const u64 nt = (ngrp + gpt - 1) / gpt;
    for (u64 item = blockIdx.x; item < nt * a.nkc; item += gridDim.x) {
        const u64 tile = item / a.nkc;
        const u32 kbeg = (u32)(item % a.nkc) * a.kchunk, kend = kbeg + a.kchunk < a.w ? kbeg + a.kchunk : a.w;
        const u64 grp = tile * gpt + gi, i0 = grp * 8;
        const bool actg = ro < a.rps && grp < ngrp;      // the same in lane 63 as in lane 62
        const u64 nvg = actg ? a.N : 0;
        u64 cpub[8], rho_o[8], rho_n[8];
        {
            u64 uo[8], un[8];
            ld8(own_of(a.u, p), i0, nvg, uo); ld8(nxt_of(a.u, p), i0, nvg, un);
            // the column ranges of one tile (and the adjacent columns of a step) replay the same
            // opening; it is counted once
            E.template open_rows<ISSUE>(op, i0, uo, un, cpub, rho_o, rho_n, kbeg == 0 && ro == 0 ? 64u * live8(i0, nvg) : 0u);
#pragma unroll
            for (int s = 0; s < 8; s++) cpub[s] -= a.base;
            if (IN_LDS) {
                wave_sync();
#pragma unroll
                for (int j = 0; j < 4; j++) {
                    s_rho[j * GT_LANES + W.m] = make_ulonglong2(rho_o[2 * j], rho_o[2 * j + 1]);
                    s_open[j * GT_TP + W.t] = make_ulonglong2(cpub[2 * j], cpub[2 * j + 1]);
                }
                wave_sync();
            }
        }
        const u64 *w1o = nullptr, *w1n = nullptr, *xto = nullptr, *xtn = nullptr;
        if (MODE == GM_COMMON) { w1o = own_of(a.W1, p) + a.w1off; w1n = nxt_of(a.W1, p) + a.w1off; }
        if (MODE == GM_ROWS) { const u64 g0 = (grp < ngrp ? grp : ngrp - 1) * 8; xto = own_of(a.XT, p) + g0; xtn = nxt_of(a.XT, p) + g0; }
        // GM_ROWS: the samples' own values of a column, fetched a whole step ahead (HBM latency)
        u64 xo[8], xn[8];
        const auto fetch_x = [&](u32 k) {              // whole groups: rows are padded to N8 and start at multiples of 64 bytes
            ld8_whole(xto + (u64)k * a.N8, xo); ld8_whole(xtn + (u64)k * a.N8, xn);
        };
        if (MODE == GM_ROWS) fetch_x(kbeg);
        u64 acc[8], acc2[8];
#pragma unroll
        for (int s = 0; s < 8; s++) { acc[s] = 0; acc2[s] = 0; }
        for (u32 k0 = kbeg; k0 < kend; k0 += a.rps) {
            const bool act = MODE == GM_STORE ? actg && k0 + ro < kend : actg;
            const u32 k = MODE == GM_STORE ? (act ? k0 + ro : kbeg) : k0;   // this lane's column (an existing one when idle)
            const u64 nv = act ? a.N : 0;              // samples of this lane that exist
            const u32 nl = live8(i0, nv);              // how many of the lane's eight tests exist
            u32 go = 0, gn = 0;
            if (HAS_G) { const Sh gk = ld(a.g, p, k); go = 0u - ((u32)gk.o & 1); gn = 0u - ((u32)gk.n & 1); }
            Sh Wk = { 0, 0 }, Wk2 = { 0, 0 };
            const u32 f = E.template tests<HAS_G, ISSUE>(op, (u64)k * ngrp + grp, [&](int h, u64 (&cd)[4], u64 (&ro)[4], u64 (&rn)[4]) {
                if (IN_LDS) {
#pragma unroll
                    for (int j = 0; j < 2; j++) {
                        const ulonglong2 c = s_open[(h / 2 + j) * GT_TP + W.t], o = s_rho[(h / 2 + j) * GT_LANES + W.m], n = s_rho[(h / 2 + j) * GT_LANES + W.nx];
                        cd[2 * j] = c.x - k; cd[2 * j + 1] = c.y - k; ro[2 * j] = o.x; ro[2 * j + 1] = o.y; rn[2 * j] = n.x; rn[2 * j + 1] = n.y;
                    }
                } else {
#pragma unroll
                    for (int j = 0; j < 4; j++) { cd[j] = cpub[h + j] - k; ro[j] = rho_o[h + j]; rn[j] = rho_n[h + j]; }
                }
            }, go, gn, nl, [&]() {
                if (MODE == GM_COMMON) { Wk.o = w1o[k]; Wk.n = w1n[k]; }
                if (MODE == GM_COMMON && NDOT == 2) Wk2 = ld(a.W2, p, a.w2off + k);
            });
            // without this the compiler adds own + next of the values right behind their loads and waits for these at the start of
            // the step (6,495 rows x 248 columns, a wavefront per SIMD: 37.4 us, 33.3 with it)
            if (MODE == GM_ROWS && ISSUE == PRF_ALONE) __builtin_amdgcn_sched_barrier(0);
            if (MODE == GM_COMMON) {
                // E W = f ? c - z : z with z = b W, c = (the public 1) W, a constant of the column:
                // ((z + (m & ~c)) xor m)
                const u64 S = Wk.o + Wk.n, nc = ~(one.o * S + one.n * Wk.o);
                const u64 S2 = Wk2.o + Wk2.n, nc2 = ~(one.o * S2 + one.n * Wk2.o);
#pragma unroll
                for (int s = 0; s < 8; s++) {
                    const u32 m = (u32)((int)(f << (31 - eq_pos(s))) >> 31);
                    const u64 mm = (u64)m | ((u64)m << 32), bo = E.row(p, s), bn = E.row(W.pn, s);
                    acc[s] += ((mm & nc) + bo * S + bn * Wk.o) ^ mm;
                    if (NDOT == 2) acc2[s] += ((mm & nc2) + bo * S2 + bn * Wk2.o) ^ mm;
                }
            } else {
                u64 Eo[8], Es[8];
#pragma unroll
                for (int s = 0; s < 8; s++) {
                    const u32 m = (u32)((int)(f << (31 - eq_pos(s))) >> 31);
                    const u64 eo = eq_select(E.row(p, s), m, k1o);
                    if (MODE == GM_STORE) {
                        Eo[s] = i0 + s < nv ? eo : 0;
                        if (a.sums) Es[s] = i0 + s < nv ? eo + eq_select(E.row(W.pn, s), m, k1n) : 0;
                    }
                    if (MODE == GM_ROWS) {
                        const Sh e = { eo, eq_select(E.row(W.pn, s), m, k1n) }, x = { xo[s], xn[s] };
                        acc[s] += prod3(e, x);
                    }
                }
                if (MODE == GM_ROWS) fetch_x(k0 + 1 < kend ? k0 + 1 : k0);
                if (MODE == GM_STORE && act && W.real) {
                    store_limbs8(p == 0 ? a.L.m[0] : (p == 1 ? a.L.m[1] : a.L.m[2]), k, i0, Eo);
                    if (a.sums) store_limbs8(p == 0 ? a.S.m[0] : (p == 1 ? a.S.m[1] : a.S.m[2]), k, i0, Es);
                }
            }
        }
        if (MODE != GM_STORE && a.nkc > 1) {
            // partial sums by atomic adds, handed round so that the lanes of a party add to consecutive
            // words (a party's 168 sums are consecutive in memory; with the eight of a lane added one
            // after the other every lane of an instruction touched a line of its own)
#pragma unroll
            for (int q = 0; q < NDOT; q++) {
                u64 *lin = s_rows;                     // 512 words
                wave_sync();
#pragma unroll
                for (int s = 0; s < 8; s++) lin[W.m * 8 + s] = q ? acc2[s] : acc[s];
                wave_sync();
                const u64 first = tile * gpt * 8;
                u64 *d = a.dacc + (u64)(3 * q + p) * a.N8 + first;
#pragma unroll
                for (int j = 0; j < 8; j++) {
                    const u32 w = j * GT_TP + W.t;
                    const u64 v = lin[GT_TP * 8 * p + w];
                    if (W.real && first + w < a.N) atomicAdd((unsigned long long *)&d[w], (unsigned long long)v);
                }
            }
        }
        if (MODE != GM_STORE && a.nkc == 1) {
#pragma unroll
            for (int q = 0; q < NDOT; q++) {
                u64 ao[8], an[8], snd[8], rcv[8];
                chacha8(E.own, grp, op, 2 + q, ao);
                W.pass64<8>(ao, an, W.nx);             // the words under the next key, from the other holder of that key
#pragma unroll
                for (int s = 0; s < 8; s++) snd[s] = (q ? acc2[s] : acc[s]) + (ao[s] - an[s]);
                W.reshare64<8>(snd, rcv);
                W.nresh += 64u * live8(i0, nvg);
#pragma unroll
                for (int s = 0; s < 8; s++)
                    if (W.real && i0 + s < nvg) {
                        Sh z = { snd[s], rcv[s] };
                        if (q == 0 && a.epi == 1) z = scale(ld(a.prev, p, i0 + s), 2) + z + one;
                        st(q ? a.out2 : a.out, p, i0 + s, z);
                    }
            }
        }
        W.drain();
    }
    W.flush(a.c.wire);
}

// ---------------------------------------------------------------------------------
// Small per-element protocols, one element per lane.

// a wavefront of an element kernel: tiles of GT_EL elements, grid-stride; every lane of the wavefront
// runs the same tiles.  LDS per wavefront: messages, material, counters.
#define GT_EL_SHARED(NS, ISSUE)                                                                \
    __shared__ uint4 s_msg[GT_LANES];                                                       \
    __shared__ u64 s_mat[GT_EL_WORDS(NS)];                                                  \
    __shared__ u64 s_cnt[6];                                                                \
    typename ElWire<ISSUE>::T W; W.init(s_msg, s_cnt);                                      \
    const int p = W.p;                                                                      \
    ElTile<NS, ISSUE> T; T.init(a.c.keys, W, s_mat);
#define GT_FOR_EL(n) for (u64 tile_ = blockIdx.x, ntiles_ = ((u64)(n) + GT_EL - 1) / GT_EL; tile_ < ntiles_; tile_ += gridDim.x)
__device__ __forceinline__ u32 el_live(u64 e0, u64 n) { return n - e0 < GT_EL ? (u32)(n - e0) : GT_EL; }

// z = B2A([x - y_pub == 0]) or the Boolean bit (BOOL_OUT).  300,007 elements: 51 us with a party per
// wavefront, 23 us in the wavefront model, 20 with the issue priorities of PRF_PAIR.
struct EqArgs { KCommon c; P6 x; const u64 *ypub; u64 ysub; P6 z; u64 n, xoff; };
template <bool BOOL_OUT, class WireT, class TileT>
__device__ __forceinline__ void eq_tile(const EqArgs &a, WireT &W, TileT &T, u64 tile)
{
    const int p = W.p;
    const u64 e0 = tile * GT_EL, e = e0 + W.t;
    const bool act = W.t < GT_EL && e < a.n;
    Sh v = { 0, 0 };
    if (act) v = ld(a.x, p, a.xoff + e) - pub(p, a.ysub + (a.ypub ? a.ypub[e] : 0));
    T.deal_mask(W, a.c.op, e0, 1, el_live(e0, a.n));
    const Dealer D = T.dealer(W);
    Sh b = eq_bit_mask(W, p, v, D, T.zb(W, 0, (u32)(e0 & 7) + W.t), act);
    if (!BOOL_OUT) b = b2a(W, p, b, D, act);
    if (act && W.real) st(a.z, p, e, b);
    W.drain();
}
template <bool BOOL_OUT>
__global__ __launch_bounds__(64) void k_eq(EqArgs a)
{
    GT_EL_SHARED(1, BOOL_OUT ? PRF_ALONE : PRF_PAIR)
    GT_FOR_EL(a.n) eq_tile<BOOL_OUT>(a, W, T, tile_);
    W.flush(a.c.wire);
}

// Bits s (own ro, next rn, in bits 0 and 16) of a lane's two elements to arithmetic sharings: one message for both.
__device__ __forceinline__ void b2a2(WWire &W, u32 ro, u32 rn, const Dealer (&D)[2], u32 na, Sh (&z)[2])
{
    u32 fo[1] = { ro ^ (D[0].bBo | (D[1].bBo << 16)) }, fr[1];
    W.pass<1>(fo, fr, W.pv);
    W.nopen += na;
    const u32 f = fo[0] ^ rn ^ (D[0].bBn | (D[1].bBn << 16)) ^ fr[0];
    const Sh one = pub(W.p, 1);
#pragma unroll
    for (int h = 0; h < 2; h++) {
        const bool set = (f >> (16 * h)) & 1;
        z[h].o = set ? one.o - D[h].bA.o : D[h].bA.o;
        z[h].n = set ? one.n - D[h].bA.n : D[h].bA.n;
    }
}

// k_eq<false> on tiles of 40 elements, two per lane (see ElPair), from as many on as there are SIMDs: the block function is two thirds of
// the work, and a pass of it yields twice the elements.  60,000 elements 9.6 us in tiles of 20, 9.0 so; 300,007 21.3 and 18.3; 2,000,000 86 and 69; but
// 30,000 8.0 and 8.1, 21,000 7.6 and 7.8.  (Order tests, 32 elements on 16 of 21 lanes a party: 300,007 24.3 and 26.4.)
__global__ __launch_bounds__(64) void k_eq_pair(EqArgs a)
{
    __shared__ uint4 s_msg[GT_LANES];
    __shared__ u64 s_mat[ElPair<40, 1>::WORDS];
    __shared__ u64 s_cnt[6];
    WWire W; W.init(s_msg, s_cnt);
    const int p = W.p;
    ElPair<40, 1> T; T.keys = a.c.keys; T.mat = s_mat;
    for (u64 tile = blockIdx.x; tile < (a.n + 39) / 40; tile += gridDim.x) {
        const u64 e0 = tile * 40;
        const u32 nel = a.n - e0 < 40 ? (u32)(a.n - e0) : 40, t = W.t < 20 ? W.t : 19, e[2] = { t, t + 20 };
        const bool act[2] = { W.t < 20 && e[0] < nel, W.t < 20 && e[1] < nel };
        const u32 na = (u32)act[0] + (u32)act[1];
        Sh v[2] = { { 0, 0 }, { 0, 0 } }, z[2];
#pragma unroll
        for (int h = 0; h < 2; h++)
            if (act[h]) v[h] = ld(a.x, p, a.xoff + e0 + e[h]) - pub(p, a.ysub + (a.ypub ? a.ypub[e0 + e[h]] : 0));
        const u32 st1[1] = { 1 };
        T.deal(W, a.c.op, e0, st1, nel);
        const Dealer D[2] = { T.dealer(W, e[0]), T.dealer(W, e[1]) };
        const u64 A[2] = { T.zb(W, 0, e[0]), T.zb(W, 0, e[1]) };
        u32 ro, rn;
        eq_bits2(W, v, D, A, na, ro, rn);
        b2a2(W, ro, rn, D, na, z);
#pragma unroll
        for (int h = 0; h < 2; h++) if (act[h] && W.real) st(a.z, p, e0 + e[h], z[h]);
        W.drain();
    }
    W.flush(a.c.wire);
}

// Completion of split inner products: z_p = partial sum + alpha (stream 2, second
// output stream 3), reshare, epilogue as in k_eqgrid.  Rows in the lanes of the element kernels:
// consecutive rows in consecutive lanes (eight rows per lane of 64 took 11 us for 48,842 rows).  The workgroups from finblk on
// run equality tests that do not depend on it (a level's leaf flags; a launch of 5 us before).
__global__ __launch_bounds__(64) void k_dot_fin(GridArgs a, u32 finblk, EqArgs eq)
{
    __shared__ uint4 s_msg[GT_LANES];
    __shared__ u64 s_mat[GT_EL_WORDS(2)];
    __shared__ u64 s_cnt[6];
    ElWire<PRF_ALONE>::T W; W.init(s_msg, s_cnt);
    const int p = W.p;
    ElTile<2> T; T.init(a.c.keys, W, s_mat);
    const Sh one = pub(p, 1);
    if (blockIdx.x >= finblk) {
        for (u64 tile = blockIdx.x - finblk; tile < (eq.n + GT_EL - 1) / GT_EL; tile += gridDim.x - finblk) eq_tile<true>(eq, W, T, tile);
        W.flush(eq.c.wire);
        return;
    }
    for (u64 tile_ = blockIdx.x; tile_ < (a.N + GT_EL - 1) / GT_EL; tile_ += finblk) {
        const u64 e0 = tile_ * GT_EL, i = e0 + W.t;
        const bool act = W.t < GT_EL && i < a.N;
        const u32 st2[2] = { 2, 3 }, w = (u32)(e0 & 7) + W.t;
        u64 part[2] = { 0, 0 };
        if (act)
            for (int q = 0; q < a.ndot; q++) part[q] = a.dacc[(u64)(3 * q + p) * a.N8 + i];
        T.deal(W, a.c.op, e0, st2, 0);
        if (act)                                       // leave zero for the next grid
            for (int q = 0; q < a.ndot; q++) a.dacc[(u64)(3 * q + p) * a.N8 + i] = 0;
        for (int q = 0; q < a.ndot; q++) {
            Sh z;
            z.o = part[q] + T.za(W, q, w);
            z.n = W.reshare1(z.o, act ? 64u : 0u);
            if (act && W.real) {
                if (q == 0 && a.epi == 1) z = scale(ld(a.prev, p, i), 2) + z + one;
                st(q == 0 ? a.out : a.out2, p, i, z);
            }
        }
        W.drain();
    }
    W.flush(a.c.wire);
}

// z = B2A([x >= y]).  300,007 elements: 54 us with a party per wavefront, 27 us in the wavefront model, 25 with the issue
// priorities of PRF_PAIR.
struct GeArgs { KCommon c; P6 x, y, z; u64 n; };
__global__ __launch_bounds__(64) void k_ge(GeArgs a)
{
    GT_EL_SHARED(2, PRF_PAIR)
    GT_FOR_EL(a.n) {
        const u64 e0 = tile_ * GT_EL, e = e0 + W.t;
        const bool act = W.t < GT_EL && e < a.n;
        Sh v = { 0, 0 };
        if (act) v = ld(a.x, p, e) - ld(a.y, p, e);
        const u32 st2[2] = { 1, 2 }, w = (u32)(e0 & 7) + W.t;
        T.deal(W, a.c.op, e0, st2, el_live(e0, a.n));
        const Dealer D = T.dealer(W);
        const Sh b = b2a(W, p, ge_bit_masks(W, p, v, D, T.zb(W, 0, w), T.zb(W, 1, w), act), D, act);
        if (act && W.real) st(a.z, p, e, b);
        W.drain();
    }
    W.flush(a.c.wire);
}

// Inference, threshold mode: bit = [x > theta]; Tidx <- 2 Tidx + bit + 1.
struct CmpArgs { KCommon c; P6 th, x, tidx; u64 n; };
__global__ __launch_bounds__(192) void k_cmp_step(CmpArgs a)
{
    const int p = party_of_wave();
    __shared__ u64 s_wire[GT_LWIRE_WORDS];
    __shared__ u64 s_cnt[6];
    Wire W; W.init(s_wire, s_cnt);
    __shared__ u64 s_prf[3][GT_PRF_SCRATCH_WORDS];
    const PartyKeys K = load_party_keys(a.c.keys, p, s_prf[p]);
    GT_FOR_TILES(a.n) {
        const u64 e = GT_ELEM();
        const bool act = e < a.n;
        Sh v = { 0, 0 };
        if (act) v = ld(a.th, p, e) - ld(a.x, p, e);
        const Dealer D = dealer_of(K, p, a.c.op, e);
        Sh b = b2a(W, p, not_bit(p, ge_bit(W, K, p, a.c.op, e, v, D, act)), D, act);
        if (act) st(a.tidx, p, e, scale(ld(a.tidx, p, e), 2) + b + pub(p, 1));
    }
    W.flush(a.c.wire);
}

// Restoring division, all steps of an element in one launch (the steps of different
// elements do not interact): step t uses operation id op + t; b = [r >= Q]; r <- r - b Q;
// quo <- 2 quo + b; r starts as S and is doubled between steps.  T: the step's material, a tile or a lane's words of it.
struct DivWords {                                      // a lane's words of a step, loaded
    Dealer D;
    u64 g, e, a;
    template <class TileT> __device__ __forceinline__ void load(const WWire &W, const TileT &T, u32 w)
    { D = T.dealer(W); g = T.zb(W, 0, w); e = T.zb(W, 1, w); a = T.za(W, 2, w); }
    __device__ __forceinline__ const Dealer &dealer(const WWire &) const { return D; }
    __device__ __forceinline__ u64 zb(const WWire &, int i, u32) const { return i == 0 ? g : e; }
    __device__ __forceinline__ u64 za(const WWire &, int, u32) const { return a; }
};
template <class WireT, class TileT>
__device__ __forceinline__ void div_step(WireT &W, const TileT &T, int p, u32 w, bool first, Sh Q, Sh &r, Sh &quo, bool act)
{
    if (!first) r = scale(r, 2);
    const Dealer D = T.dealer(W);
    const Sh b = b2a(W, p, ge_bit_masks(W, p, r - Q, D, T.zb(W, 0, w), T.zb(W, 1, w), act), D, act);
    const Sh bq = mult_sh(W, b, Q, T.za(W, 2, w), act);
    r = r - bq;
    quo = scale(quo, 2) + b;
}
// Material of all steps of a division by NW wavefronts side by side, then the steps by the first of
// them: with few elements the steps' PRF blocks would otherwise lie in the chain, one per step.
// NW = 1: a slot that is dealt anew before every step.
template <int NW, class WireT, class TileT>
__device__ __forceinline__ void div_steps_el(WireT &W, TileT &T, u64 *s_mat, int p, u32 op, u64 e0, u32 nel, u32 nsteps, Sh Q, Sh &r, Sh &quo, bool act)
{
    const u32 st3[3] = { 1, 2, 3 }, w = (u32)(e0 & 7) + W.t;
    if (NW > 1) {
        for (u32 t = threadIdx.x / GT_LANES; t < nsteps; t += NW) { T.mat = s_mat + t * GT_EL_WORDS(3); T.deal(W, op + t, e0, st3, nel); }
        __syncthreads();
    }
    if (NW == 1)
        for (u32 t = 0; t < nsteps; t++) {
            T.deal(W, op + t, e0, st3, nel);
            div_step(W, T, p, w, t == 0, Q, r, quo, act);
        }
    else if (threadIdx.x < GT_LANES) {
        // a chain: the next step's words are loaded during a step (scores of 267 x 22 24.5 us a level, 23.5 so)
        T.mat = s_mat;
        DivWords next;
        next.load(W, T, w);
        for (u32 t = 0; t < nsteps; t++) {
            const DivWords m = next;
            T.mat = s_mat + (t + 1 < nsteps ? t + 1 : t) * GT_EL_WORDS(3);
            next.load(W, T, w);
            div_step(W, m, p, w, t == 0, Q, r, quo, act);
        }
    }
    if (NW > 1) __syncthreads();                       // the material is dealt anew for the next tile
}
#define GT_DIV_STEPS 21                                // GT_MAX_TAU + 1
#define GT_DIV_SHARED(NW)                                                                  \
    __shared__ uint4 s_msg[NW][GT_LANES];                                                   \
    __shared__ u64 s_mat[(NW > 1 ? GT_DIV_STEPS : 1) * GT_EL_WORDS(3)];                      \
    __shared__ u64 s_cnt[NW][6];                                                            \
    const u32 wave_ = __builtin_amdgcn_readfirstlane(threadIdx.x / GT_LANES);               \
    typename ElWire<NW == 1 ? PRF_PAIR : PRF_ALONE>::T W; W.init(s_msg[wave_], s_cnt[wave_]); \
    const int p = W.p;                                                                      \
    ElTile<3, NW == 1 ? PRF_PAIR : PRF_ALONE> T; T.init(a.c.keys, W, s_mat);

// 100,003 quotients, 17 steps: 304 us with a party per wavefront, 109 us in the wavefront model, 75 with the issue priorities of
// PRF_PAIR (VALU: a PRF pass and 240 instructions of protocol per step and 20 elements).
struct DivArgs { KCommon c; P6 S, Q, quo; u64 n; u32 nsteps; };
template <int NW>
__global__ __launch_bounds__(64 * NW) void k_div(DivArgs a)
{
    GT_DIV_SHARED(NW)
    GT_FOR_EL(a.n) {
        const u64 e0 = tile_ * GT_EL, e = e0 + W.t;
        const bool act = W.t < GT_EL && e < a.n;
        Sh r = { 0, 0 }, Q = { 0, 0 }, quo = { 0, 0 };
        if (act) { Q = ld(a.Q, p, e); r = ld(a.S, p, e); }
        div_steps_el<NW>(W, T, s_mat, p, a.c.op, e0, el_live(e0, a.n), a.nsteps, Q, r, quo, act);
        if (act && W.real && wave_ == 0) st(a.quo, p, e, quo);
        W.drain();
    }
    W.flush(a.c.wire);
}

// Gini scores of a level in one launch (Sec. V-B, Eq. (1)).  Element q = (r*d+k)*2 + j:
//   op:          S = sum_c n_jc^2, Q = n_j * n with n_1c = C[r][k*K+c], n_0c = tot_c - n_1c
//   op+1:        Q <- Q + [Q == 0] (empty branch: divisor 1)
//   op+2 ..:     restoring division, tau+1 steps
//   op+tau+3:    score = quo(j=0) + quo(j=1), masked = score * gamma[r*d+k], written to `score`
// Everything is local to the two elements of a candidate, so nothing but the masked score reaches memory
// (five launches and six arrays before; 17 steps for up to 9,408 elements 24 us, 105 us before).
struct ScoreArgs { KCommon c; P6 C, gamma, score; u64 n; u32 d, K, CW, nsteps; };
template <int NW>
__global__ __launch_bounds__(64 * NW) void k_score(ScoreArgs a)
{
    GT_DIV_SHARED(NW)
    const u64 dK = (u64)a.d * a.K;
    GT_FOR_EL(a.n) {
        const u64 e0 = tile_ * GT_EL, q = e0 + W.t, cand = q / 2;
        const bool act = W.t < GT_EL && q < a.n;
        const u32 nel = el_live(e0, a.n), w = (u32)(e0 & 7) + W.t;
        const u32 cb = wave_ == 0 ? 1u : 0u;           // every wavefront runs the head of the tile (it is short), one counts
        Sh nj = { 0, 0 }, n = { 0, 0 }, S, Q, quo = { 0, 0 };
        u64 s = 0;
        if (act) {
            const u64 r = cand / a.d, k = cand % a.d, br = q & 1;
            for (u32 cl = 0; cl < a.K; cl++) {
                const Sh n1 = ld(a.C, p, r * a.CW + k * a.K + cl), tot = ld(a.C, p, r * a.CW + dK + cl);
                const Sh njc = br ? n1 : tot - n1;
                nj = nj + njc; n = n + tot;
                s += prod3(njc, njc);
            }
        }
        T.mat = s_mat + (NW > 1 ? wave_ : 0u) * GT_EL_WORDS(3);
        {
            const u32 sn[3] = { 0, 1, 1 };
            T.deal(W, a.c.op, e0, sn, 0);
            u64 snd[2] = { s + T.za(W, 0, w), prod3(nj, n) + T.za(W, 1, w) }, rcv[2];
            W.template reshare<2>(snd, rcv, act ? 128u * cb : 0u);
            S.o = snd[0]; S.n = rcv[0]; Q.o = snd[1]; Q.n = rcv[1];
        }
        const bool actc = act && cb;
        {
            const u32 sn[3] = { 1, 1, 1 };
            T.deal(W, a.c.op + 1, e0, sn, nel);
            const Dealer D = T.dealer(W);
            Q = Q + b2a(W, p, eq_bit_mask(W, p, Q, D, T.zb(W, 0, w), actc), D, actc);
        }
        if (NW > 1) __syncthreads();                   // the head's material of all wavefronts has been read
        div_steps_el<NW>(W, T, s_mat, p, a.c.op + 2, e0, nel, a.nsteps, Q, S, quo, actc);
        if (wave_ == 0) {
            // the candidate's two quotients meet in its even lane (the party's own words, no message)
            const u64 mine[2] = { quo.o, quo.n };
            u64 other[2];
            W.template pass64<2>(mine, other, W.lane_of(W.t < GT_EL ? W.t ^ 1 : W.t));
            const bool ev = act && !(W.t & 1);
            Sh sc = { quo.o + other[0], quo.n + other[1] }, g = { 0, 0 };
            if (ev) g = ld(a.gamma, p, cand);
            const u32 sn[3] = { 0, 0, 0 };
            T.mat = s_mat;
            T.deal(W, a.c.op + 2 + a.nsteps, e0 / 2, sn, 0);
            const Sh z = mult_sh(W, sc, g, T.za(W, 0, (u32)((e0 / 2) & 7) + W.t / 2), ev);
            if (ev && W.real) st(a.score, p, cand, z);
        }
        if (NW > 1) __syncthreads();
        W.drain();
    }
    W.flush(a.c.wire);
}

// Compare-and-select of a tile: b = [right > left]; val = left + b (right-left); idx likewise (material
// of operation `op`, elements from e0).
template <class WireT, class TileT>
__device__ __forceinline__ void select_el(WireT &W, TileT &T, int p, u32 op, u64 e0, u32 nel, Sh &L, Sh R, Sh &IL, Sh IR, bool act)
{
    const u32 st4[4] = { 1, 2, 3, 4 }, w = (u32)(e0 & 7) + W.t;
    T.deal(W, op, e0, st4, nel);
    const Dealer D = T.dealer(W);
    const Sh b = b2a(W, p, not_bit(p, ge_bit_masks(W, p, L - R, D, T.zb(W, 0, w), T.zb(W, 1, w), act)), D, act);
    u64 snd[2] = { prod3(b, R - L) + T.za(W, 2, w), prod3(b, IR - IL) + T.za(W, 3, w) }, rcv[2];
    W.template reshare<2>(snd, rcv, act ? 128u : 0u);
    L.o += snd[0]; L.n += rcv[0]; IL.o += snd[1]; IL.n += rcv[1];
}

// The tournament of a level's masked scores.  Round l (operation op + l) compares arrays of length
// P2 >> l, node after node: element e = r*half + m, left 2e, right 2e + 1 of the round before; the scores
// are padded with 0, the indices start as k.
struct SelectPair { Sh L, R, IL, IR; };
// element e of the first round (half = 1 << lgh)
__device__ __forceinline__ SelectPair first_pair(const P6 &score, int p, u64 e, u32 lgh, u32 d)
{
    const u64 r = e >> lgh;
    const u32 k = 2 * (u32)(e - (r << lgh));
    SelectPair q = { { 0, 0 }, { 0, 0 }, pub(p, k), pub(p, k + 1) };
    if (k < d) q.L = ld(score, p, r * d + k);
    if (k + 1 < d) q.R = ld(score, p, r * d + k + 1);
    return q;
}
__device__ __forceinline__ SelectPair next_pair(const P6 &val, const P6 &idx, int p, u64 e)
{
    SelectPair q = { ld(val, p, 2 * e), ld(val, p, 2 * e + 1), ld(idx, p, 2 * e), ld(idx, p, 2 * e + 1) };
    return q;
}

// One round of all nodes, tiles of GT_EL elements over the whole chip, for rounds that fill it.
struct SelectArgs { KCommon c; P6 score, vin, iin, vout, iout; u64 n; u32 d, lgh; int first; };
__global__ __launch_bounds__(64) void k_select_round(SelectArgs a)
{
    GT_EL_SHARED(4, PRF_PAIR)
    GT_FOR_EL(a.n) {
        const u64 e0 = tile_ * GT_EL, e = e0 + W.t;
        const bool act = W.t < GT_EL && e < a.n;
        SelectPair q = { { 0, 0 }, { 0, 0 }, { 0, 0 }, { 0, 0 } };
        if (act) q = a.first ? first_pair(a.score, p, e, a.lgh, a.d) : next_pair(a.vin, a.iin, p, e);
        select_el(W, T, p, a.c.op, e0, el_live(e0, a.n), q.L, q.R, q.IL, q.IR, act);
        if (act && W.real) { st(a.vout, p, e, q.L); st(a.iout, p, e, q.IL); }
        W.drain();
    }
    W.flush(a.c.wire);
}

// All rounds from arrays of `len` on in one launch: NW wavefronts per node, tiles of 16 elements
// ((e0 mod 8) + 16 <= 24 for any e0), the rounds' results in LDS.  One wavefront holds the 32/len nodes
// whose first rounds make up a tile and needs no barrier; with two, four or eight a node's first round is a
// tile per wavefront (two for len = 512) and a barrier ends a round.  LDS per wavefront 7 KB (10 with eight).
// Bound: the chain of the rounds (about 3 us each) and, from thousands of nodes on, the vector ALU.  One node of 512
// candidates 27 us; 4,096 nodes of 8 candidates 11 us, where a workgroup of eight wavefronts and 90 KB for every node
// took 126 and a launch per round 40; 32,768 nodes 40 us (884; 82).
#define GT_ARGMAX_LDS 512
struct ArgmaxArgs { KCommon c; P6 score, vin, iin, SD; u64 nh; u32 d, len, lgh; int first; };   // lgh: log2(len / 2); first: from the scores, else from vin, iin
template <int NW>
__global__ __launch_bounds__(64 * NW) void k_argmax(ArgmaxArgs a)
{
    constexpr u32 RES = NW == 8 ? GT_ARGMAX_LDS / 2 : 16 * NW;          // elements of the first round
    __shared__ uint4 s_msg[NW][GT_LANES];
    __shared__ u64 s_mat[NW][GT_EL_WORDS(4)];
    __shared__ u64 s_cnt[NW][6];
    __shared__ u64 s_buf[12][RES + RES / 2];                            // results of the even rounds, of the odd ones
    const u32 wave = __builtin_amdgcn_readfirstlane(threadIdx.x / GT_LANES);
    ElWire<PRF_ALONE>::T W; W.init(s_msg[wave], s_cnt[wave]);
    const int p = W.p;
    ElTile<4> T; T.init(a.c.keys, W, s_mat[wave]);
    u64 *vo = s_buf[4 * p], *vn = s_buf[4 * p + 1], *io = s_buf[4 * p + 2], *in = s_buf[4 * p + 3];
    const u32 per = NW == 1 ? 32 / a.len : 1;                           // nodes of a workgroup
    for (u64 r0 = (u64)blockIdx.x * per; r0 < a.nh; r0 += (u64)gridDim.x * per) {
        const u32 nn = a.nh - r0 < per ? (u32)(a.nh - r0) : per;
        u32 round = 0, from = RES, to = 0;
        for (u32 half = a.len / 2; half > 0; half /= 2, round++) {
            const u32 n = nn * half;
            for (u32 m0 = wave * 16; m0 < n; m0 += NW * 16) {
                const u32 nel = n - m0 < 16 ? n - m0 : 16, m = m0 + W.t;
                const bool act = W.t < nel;
                SelectPair q = { { 0, 0 }, { 0, 0 }, { 0, 0 }, { 0, 0 } };
                if (act) {
                    if (round > 0) {
                        const u32 j = from + 2 * m;
                        q = { { vo[j], vn[j] }, { vo[j + 1], vn[j + 1] }, { io[j], in[j] }, { io[j + 1], in[j + 1] } };
                    } else q = a.first ? first_pair(a.score, p, (r0 << a.lgh) + m, a.lgh, a.d) : next_pair(a.vin, a.iin, p, (r0 << a.lgh) + m);
                }
                select_el(W, T, p, a.c.op + round, r0 * half + m0, nel, q.L, q.R, q.IL, q.IR, act);
                if (act && W.real) {
                    if (half == 1) st(a.SD, p, r0 + m, q.IL);
                    else { vo[to + m] = q.L.o; vn[to + m] = q.L.n; io[to + m] = q.IL.o; in[to + m] = q.IL.n; }
                }
            }
            from = to; to = RES - to;
            if (NW > 1) __syncthreads(); else wave_sync();
        }
        if (a.len == 1)                                                 // one candidate: index 0
            for (u32 j = W.t; j < nn; j += GT_EL) if (W.real && wave == 0) st(a.SD, p, r0 + j, Sh{ 0, 0 });
        W.drain();
    }
    W.flush(a.c.wire);
}

// Label = first maximum of the class totals, the K-1 selections of a node in one launch (operation
// op + cl - 1): left starts as class 0, right = class cl with the index constant cl.
struct LabelArgs { KCommon c; P6 C, lab; u64 n, dK, laboff; u32 K, CW; };
__global__ __launch_bounds__(64) void k_labels(LabelArgs a)
{
    GT_EL_SHARED(4, PRF_ALONE)
    GT_FOR_EL(a.n) {
        const u64 e0 = tile_ * GT_EL, e = e0 + W.t;
        const bool act = W.t < GT_EL && e < a.n;
        Sh L = { 0, 0 }, IL = { 0, 0 };
        if (act) L = ld(a.C, p, e * a.CW + a.dK);
        for (u32 cl = 1; cl < a.K; cl++) {
            Sh R = { 0, 0 };
            if (act) R = ld(a.C, p, e * a.CW + a.dK + cl);
            select_el(W, T, p, a.c.op + cl - 1, e0, el_live(e0, a.n), L, R, IL, pub(p, cl), act);
        }
        if (act && W.real) st(a.lab, p, a.laboff + e, IL);
        W.drain();
    }
    W.flush(a.c.wire);
}

// Updates of a level in one launch, the first gblk workgroups
//   op:   gamma[r][k] <- gamma[r][k] * (1 - [SD[r] == k])
// the others, node r:
//   op+1: pure = [n^2 - sum_c tot_c^2 == 0]; split = isLeaf and not pure;
//         F[base+r] <- F (1 - split); children F <- 2 - split.
struct UpdateArgs { KCommon c; P6 SD, gamma, C, isLeaf, F, split; u64 n, base, dK; u32 d, K, CW, gblk; };
__global__ __launch_bounds__(64) void k_update(UpdateArgs a)
{
    GT_EL_SHARED(3, PRF_ALONE)
    const u32 sn[3] = { 1, 2, 3 };
    if (blockIdx.x < a.gblk) {
        const u64 n = a.n * a.d;
        for (u64 tile = blockIdx.x; tile < (n + GT_EL - 1) / GT_EL; tile += a.gblk) {
            const u64 e0 = tile * GT_EL, e = e0 + W.t;
            const bool act = W.t < GT_EL && e < n;
            const u32 w = (u32)(e0 & 7) + W.t;
            Sh v = { 0, 0 }, g = { 0, 0 };
            if (act) { v = ld(a.SD, p, e / a.d) - pub(p, e % a.d); g = ld(a.gamma, p, e); }
            T.deal(W, a.c.op, e0, sn, el_live(e0, n));
            const Dealer D = T.dealer(W);
            const Sh oh = b2a(W, p, eq_bit_mask(W, p, v, D, T.zb(W, 0, w), act), D, act);
            const Sh z = mult_sh(W, g, pub(p, 1) - oh, T.za(W, 1, w), act);
            if (act && W.real) st(a.gamma, p, e, z);
            W.drain();
        }
    } else {
        for (u64 tile = blockIdx.x - a.gblk; tile < (a.n + GT_EL - 1) / GT_EL; tile += gridDim.x - a.gblk) {
            const u64 e0 = tile * GT_EL, r = e0 + W.t;
            const bool act = W.t < GT_EL && r < a.n;
            const u32 w = (u32)(e0 & 7) + W.t;
            Sh n = { 0, 0 }, leaf = { 0, 0 }, f = { 0, 0 };
            u64 dv = 0;
            if (act) {
                for (u32 cl = 0; cl < a.K; cl++) {
                    const Sh tc = ld(a.C, p, r * a.CW + a.dK + cl);
                    n = n + tc;
                    dv -= prod3(tc, tc);
                }
                dv += prod3(n, n);
                leaf = ld(a.isLeaf, p, r);
                f = ld(a.F, p, a.base + r);
            }
            T.deal(W, a.c.op + 1, e0, sn, el_live(e0, a.n));
            const Dealer D = T.dealer(W);
            Sh d;
            d.o = dv + T.za(W, 1, w);
            d.n = W.reshare1(d.o, act ? 64u : 0u);
            const u64 A = T.zb(W, 0, w);
            const Sh npure = not_bit(p, eq_bit_mask(W, p, d, D, A, act));
            const Sh sA = b2a(W, p, and_bit(W, leaf, npure, A >> 63, act), D, act);
            const Sh keep = pub(p, 1) - sA;
            const Sh fz = mult_sh(W, f, keep, T.za(W, 2, w), act);
            if (act && W.real) {
                st(a.split, p, r, sA);
                st(a.F, p, a.base + r, fz);
                const Sh ch = keep + pub(p, 1);
                st(a.F, p, 2 * (a.base + r) + 1, ch);
                st(a.F, p, 2 * (a.base + r) + 2, ch);
            }
            W.drain();
        }
    }
    W.flush(a.c.wire);
}

// ---------------------------------------------------------------------------------
// Data partition by products with the previous level's per-sample leaf one-hot (a variant
// beyond the paper's listing: no per-sample equality tests).
//   k_onehot  : OH[r][k] = [T[base + r] == k] as an arithmetic sharing, written as limb bytes (BYTES) or as words, for k_oh_limbs
//   k_part_mm : sel[k][i] = sum_r L[r][i] * OH[r][k], zero sharing of stream 0, word k*N8+i, and
//               M[i] <- 2 M[i] + sum_k sel[k][i] * X[k][i] + 1, zero sharing of stream 0, word i
//               (gt_partmm.hpp, on the matrix cores)
// OHL[((p*2 + w)*8 + s)*dpad + k)*rpad + r] = limb s of (w ? own : own + next) of party p's OH[r][k], zero for r >= np or k >= d.  BYTES: the first
// elblk workgroups are the tests, the others zero what is padded, a row of r per thread; a launch less, but a line of OHL per byte.  Which: onehot_bytes.
struct OnehotArgs { KCommon c; P6 T, OH; unsigned char *OHL; u64 base; u32 np, d, rpad, dpad, elblk; };
template <bool BYTES>
__global__ __launch_bounds__(64) void k_onehot(OnehotArgs a)
{
    if (BYTES && blockIdx.x >= a.elblk) {
        const u64 rows = 48ull * a.dpad, step = (u64)(gridDim.x - a.elblk) * 64;
        for (u64 t = (u64)(blockIdx.x - a.elblk) * 64 + threadIdx.x; t < rows; t += step) {
            const u32 r0 = t % a.dpad < a.d ? a.np : 0;
            unsigned char *row = a.OHL + t * a.rpad;
            for (u32 r = r0; r < ((r0 + 3) & ~3u); r++) row[r] = 0;
            for (u32 r = (r0 + 3) & ~3u; r < a.rpad; r += 4) *(u32 *)(row + r) = 0;
        }
        return;
    }
    GT_EL_SHARED(1, PRF_ALONE)
    const u64 n = (u64)a.np * a.d;
    for (u64 tile_ = blockIdx.x; tile_ < (n + GT_EL - 1) / GT_EL; tile_ += a.elblk) {
        const u64 e0 = tile_ * GT_EL, e = e0 + W.t;
        const bool act = W.t < GT_EL && e < n;
        const u32 r = (u32)(e / a.d), kc = (u32)(e - (u64)r * a.d);
        Sh v = { 0, 0 };
        if (act) v = ld(a.T, p, a.base + r) - pub(p, kc);
        const u32 s1[1] = { 1 };
        T.deal(W, a.c.op, e0, s1, el_live(e0, n));
        const Dealer D = T.dealer(W);
        const Sh oh = b2a(W, p, eq_bit_mask(W, p, v, D, T.zb(W, 0, (u32)(e0 & 7) + W.t), act), D, act);
        if (!BYTES) { if (act && W.real) st(a.OH, p, e, oh); }
        else if (act && W.real) {
#pragma unroll
            for (int w = 0; w < 2; w++) {
                const u64 y = ((w ? oh.o : oh.o + oh.n) + GT_BIAS) ^ GT_BIAS;
#pragma unroll
                for (int s = 0; s < 8; s++) a.OHL[((u64)((2 * p + w) * 8 + s) * a.dpad + kc) * a.rpad + r] = (unsigned char)(y >> (8 * s));
            }
        }
        W.drain();
    }
    W.flush(a.c.wire);
}

// ---------------------------------------------------------------------------------
// The protocols as the paper prints them (Sec. V-A, Alg. "Oblivious Array Access"; Sec. V-B,
// Alg. "Oblivious Learning"), for small inputs: every array element goes through a
// SelectShare of its own - conversion of the comparison bit with the element's own daBit,
// the opened value counted as a ring element, then a product with a zero-sharing word and
// a reshare of its own - and the selected elements are added up locally (atomic adds of
// both components: exact and order-free in the ring).  One element per lane; streams 0
// dealer, 1 masks, 2 product, all indexed by the element.
struct LitOaaArgs { KCommon c; P6 u; u64 base; u32 w; u64 N, N8; P6 W1; u64 w1off; P6 XT; u64 *acc; };
template <bool ROWS>
__global__ __launch_bounds__(192) void k_oaa_literal(LitOaaArgs a)
{
    const int p = party_of_wave();
    __shared__ u64 s_wire[GT_LWIRE_WORDS];
    __shared__ u64 s_cnt[6];
    Wire W; W.init(s_wire, s_cnt);
    __shared__ u64 s_prf[3][GT_PRF_SCRATCH_WORDS];
    const PartyKeys K = load_party_keys(a.c.keys, p, s_prf[p]);
    GT_FOR_TILES((u64)a.w * a.N8) {
        const u64 e = GT_ELEM(), k = e / a.N8, i = e % a.N8;
        const bool act = k < a.w && i < a.N;
        Sh v = { 0, 0 }, wv = { 0, 0 };
        if (act) {
            v = ld(a.u, p, i) - pub(p, a.base + k);
            wv = ROWS ? ld(a.XT, p, k * a.N8 + i) : ld(a.W1, p, a.w1off + k);
        }
        const Dealer D = dealer_of(K, p, a.c.op, e);
        u64 A;
        const Sh E = b2a(W, p, eq_bit(W, K, p, a.c.op, e, v, D, A, act), D, act, 64);
        const Sh z = mult_sh(W, E, wv, zero_a(K, a.c.op, 2, e), act);
        if (act) {
            atomicAdd((unsigned long long *)&a.acc[(u64)(2 * p) * a.N8 + i], (unsigned long long)z.o);
            atomicAdd((unsigned long long *)&a.acc[(u64)(2 * p + 1) * a.N8 + i], (unsigned long long)z.n);
        }
    }
    W.flush(a.c.wire);
}

// out[i] = the sums (own, next) [epi 1: 2*prev[i] + sum + 1]; the sums are left at zero
__global__ __launch_bounds__(256) void k_lit_fin(u64 *acc, u64 N, u64 N8, P6 out, P6 prev, int epi)
{
    for (u64 i = (u64)blockIdx.x * blockDim.x + threadIdx.x; i < N; i += (u64)gridDim.x * blockDim.x)
        for (int p = 0; p < 3; p++) {
            u64 *ao = &acc[(u64)(2 * p) * N8 + i], *an = &acc[(u64)(2 * p + 1) * N8 + i];
            Sh z = { *ao, *an };
            *ao = 0; *an = 0;
            if (epi == 1) z = scale(ld(prev, p, i), 2) + z + pub(p, 1);
            st(out, p, i, z);
        }
}

// per-sample leaf flags as Boolean bits: LB[r*N8 + i] = [M[i] - base == r] and isLeaf[r]
struct LcfArgs { KCommon c; P6 M, isLeaf, LB; u64 base; u32 nh; u64 N, N8; };
__global__ __launch_bounds__(192) void k_lcf_bits(LcfArgs a)
{
    const int p = party_of_wave();
    __shared__ u64 s_wire[GT_LWIRE_WORDS];
    __shared__ u64 s_cnt[6];
    Wire W; W.init(s_wire, s_cnt);
    __shared__ u64 s_prf[3][GT_PRF_SCRATCH_WORDS];
    const PartyKeys K = load_party_keys(a.c.keys, p, s_prf[p]);
    GT_FOR_TILES((u64)a.nh * a.N8) {
        const u64 e = GT_ELEM(), r = e / a.N8, i = e % a.N8;
        const bool act = r < a.nh && i < a.N;
        Sh v = { 0, 0 }, g = { 0, 0 };
        if (act) { v = ld(a.M, p, i) - pub(p, a.base + r); g = ld(a.isLeaf, p, r); }
        const Dealer D = dealer_of(K, p, a.c.op, e);
        u64 A;
        Sh b = eq_bit(W, K, p, a.c.op, e, v, D, A, act);
        b = and_bit(W, b, g, A >> 63, act);
        if (act) st(a.LB, p, e, b);
    }
    W.flush(a.c.wire);
}

// Statistics counting element by element: e = (r*PW + q)*N8 + i, q = row*2dd + 2k + v the
// position in the (1+K) x 2dd counter array (dd = d, or 1 at the label level).
struct LitCountArgs { KCommon c; P6 LB, XT, YT; LimbSet B; LimbTri C; int comps; u64 N, N8; u32 nh, d, dd, K; u64 *acc; };
__global__ __launch_bounds__(192) void k_count_literal(LitCountArgs a)
{
    const int p = party_of_wave();
    __shared__ u64 s_wire[GT_LWIRE_WORDS];
    __shared__ u64 s_cnt[6];
    Wire W; W.init(s_wire, s_cnt);
    __shared__ u64 s_prf[3][GT_PRF_SCRATCH_WORDS];
    const PartyKeys K = load_party_keys(a.c.keys, p, s_prf[p]);
    const u64 PW = (u64)(1 + a.K) * 2 * a.dd, total = (u64)a.nh * PW * a.N8;
    GT_FOR_TILES(total) {
        const u64 e = GT_ELEM(), i = e % a.N8, rq = e / a.N8, r = rq / PW, q = rq % PW;
        const bool act = e < total && i < a.N;
        Sh s = { 0, 0 }, cv = { 0, 0 };
        if (act) {
            const u64 row = q / (2 * a.dd), k = (q % (2 * a.dd)) / 2, v = q & 1;
            const Sh x = ld(a.XT, p, k * a.N8 + i);
            if (row == 0) cv = v ? x : pub(p, 1) - x;
            else {
                const u64 col = k * a.K + (row - 1);
                Sh xy;
                if (a.comps) { xy.o = load_limbs1(a.C.m[p], col, i); xy.n = load_limbs1(a.C.m[p == 2 ? 0 : p + 1], col, i); }
                else { xy.o = load_limbs1(a.B.m[p][1], col, i); xy.n = load_limbs1(a.B.m[p][0], col, i) - xy.o; }
                cv = v ? xy : ld(a.YT, p, (row - 1) * a.N8 + i) - xy;
            }
            s = ld(a.LB, p, r * a.N8 + i);
        }
        const Dealer D = dealer_of(K, p, a.c.op, e);
        const Sh E = b2a(W, p, s, D, act, 64);
        const Sh z = mult_sh(W, E, cv, zero_a(K, a.c.op, 2, e), act);
        if (act) {
            atomicAdd((unsigned long long *)&a.acc[(u64)(2 * p) * a.nh * PW + rq], (unsigned long long)z.o);
            atomicAdd((unsigned long long *)&a.acc[(u64)(2 * p + 1) * a.nh * PW + rq], (unsigned long long)z.n);
        }
    }
    W.flush(a.c.wire);
}

// compact statistics from the accumulated counter arrays (local linear operations), added
// to the inherited ones
__global__ __launch_bounds__(256) void k_from_paper(u64 *acc, P6 C, u32 nh, u32 d, u32 dd, u32 K, u32 CW)
{
    const u64 PW = (u64)(1 + K) * 2 * dd, n = (u64)nh * K;
    for (u64 t = (u64)blockIdx.x * blockDim.x + threadIdx.x; t < n; t += (u64)gridDim.x * blockDim.x) {
        const u64 r = t / K, cl = t % K;
        for (int p = 0; p < 3; p++)
            for (int pl = 0; pl < 2; pl++) {
                u64 *o = acc + (u64)(2 * p + pl) * nh * PW + r * PW + (cl + 1) * 2 * dd;
                u64 *dst = pl ? C.n[p] : C.o[p];
                dst[r * CW + (u64)d * K + cl] += o[0] + o[1];
                if (dd == d) for (u32 k = 0; k < d; k++) dst[r * CW + (u64)k * K + cl] += o[2 * k + 1];
            }
    }
}

// ---------------------------------------------------------------------------------
// Heuristic computation by reconstruction, the host analogue of the TEE-based protocol of
// Sec. V-B: the scorer (a fourth role, not one of the parties) reconstructs the level's C,
// gamma and F from the three components and computes in the clear what the MPC protocol
// computes: fixed-point scores sum_j floor(S_j 2^tau / Q_j) (empty branch: 0) masked by
// gamma, the first maximum, the updated gamma, purity n^2 = sum_c tot_c^2, node types.
// One workgroup per node; plain results for the sharing kernel.
struct HcOpenArgs { P6 C, gamma, F; u64 base; u32 nh, d, K, CW, tau; u64 *SD, *G, *Fn, *Fc, *Sp, *SC; };
__device__ __forceinline__ u64 rec3(const P6 &a, u64 e) { return a.o[0][e] + a.n[0][e] + a.o[2][e]; }

__global__ __launch_bounds__(256) void k_hc_open(HcOpenArgs a)
{
    __shared__ u64 s_tot[16], s_best[256];
    __shared__ u32 s_idx[256];
    const u32 tid = threadIdx.x;
    const u64 dK = (u64)a.d * a.K;
    for (u32 r = blockIdx.x; r < a.nh; r += gridDim.x) {
        if (tid < a.K) s_tot[tid] = rec3(a.C, (u64)r * a.CW + dK + tid);
        __syncthreads();
        u64 n = 0;
        for (u32 cl = 0; cl < a.K; cl++) n += s_tot[cl];
        u64 best = 0; u32 bi = 0xffffffffu;
        for (u32 k = tid; k < a.d; k += blockDim.x) {
            u64 score = 0;
            for (int br = 0; br < 2; br++) {
                u64 nj = 0, S = 0;
                for (u32 cl = 0; cl < a.K; cl++) {
                    const u64 n1 = rec3(a.C, (u64)r * a.CW + (u64)k * a.K + cl);
                    const u64 njc = br ? n1 : s_tot[cl] - n1;
                    nj += njc; S += njc * njc;
                }
                u64 Q = nj * n;
                if (Q == 0) Q = 1;
                score += (S << a.tau) / Q;
            }
            const u64 g = rec3(a.gamma, (u64)r * a.d + k);
            score *= g;
            a.SC[(u64)r * a.d + k] = score; a.G[(u64)r * a.d + k] = g;
            if (bi == 0xffffffffu || score > best) { best = score; bi = k; }   // ascending k: the first maximum of this thread
        }
        s_best[tid] = best; s_idx[tid] = bi;
        __syncthreads();
        for (u32 st = 128; st > 0; st >>= 1) {         // larger score wins, then the lower index
            if (tid < st) {
                const u64 ob = s_best[tid + st]; const u32 oi = s_idx[tid + st];
                if (oi != 0xffffffffu && (s_idx[tid] == 0xffffffffu || ob > s_best[tid] || (ob == s_best[tid] && oi < s_idx[tid]))) {
                    s_best[tid] = ob; s_idx[tid] = oi;
                }
            }
            __syncthreads();
        }
        if (tid == 0) {
            const u32 sd = s_idx[0];
            u64 sq = 0;
            for (u32 cl = 0; cl < a.K; cl++) sq += s_tot[cl] * s_tot[cl];
            const u64 F = rec3(a.F, a.base + r);
            const u64 split = (F == 1 && n * n - sq != 0) ? 1 : 0;
            a.SD[r] = sd; a.G[(u64)r * a.d + sd] = 0;
            a.Sp[r] = split; a.Fn[r] = F * (1 - split); a.Fc[r] = 2 - split;
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------------
// Statistics counting as a contraction in Z_2^64 (Sec. V-B):
//   Z_p[r][col] = sum_i L_p[r][i] * (B_p + B_{p+1})[col][i] + L_{p+1}[r][i] * B_p[col][i]
//              or sum_i (L_p + L_{p+1})[r][i] * B_p[col][i] + L_p[r][i] * B_{p+1}[col][i]
// with L the per-sample leaf one-hot and B the sample-contiguous columns (XY products,
// then the K class indicators).  Both operands are uniformly random 64-bit shares, so
// this is a dense integer GEMM; it runs on the matrix cores in signed 8-bit limbs:
//   x*y mod 2^64 = sum_{s+t<=7} d_s(x) d_t(y) 256^(s+t),
// 36 limb pairs, one v_mfma_i32_32x32x32_i8 each, accumulated per u = s+t in int32.
// |d_s d_t| <= 2^14 and at most 8 pairs x 2 products x 4096 samples meet in one
// accumulator, which stays below 2^31.  A wavefront owns a 32 x 64 output tile
// (8 x 2 accumulators of 16 registers); the sample range is split over workgroups
// and the recombined 64-bit partial sums meet by atomic adds (exact, order-free).
typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
// sample blocks of 32 per workgroup: the int32 accumulators would allow 128; with 64 the launch
// has twice the workgroups to balance over the compute units and takes 3 % less time
#define CT_CHUNK_BLOCKS 64
// A[p][q] (rows: nodes) and B[p][q] (rows: columns), q = 0, 1: party p's two products
// bcol0: first column (row of B) of this launch, zcol0: its column in the output
// rt: row tiles of 32 per workgroup (4, 2 or 1); the other 4/rt wavefronts take further column tiles
// chunkblk: sample blocks of 32 per workgroup (at most CT_CHUNK_BLOCKS; the int32 accumulators bound it by 128)
// nns: slots per chunk (0 = none) for one more column group on 16-wide tiles, at most 16 columns unless x holds them (first
// column nbcol0 of B, column nzcol0 of the output), handled by the same launch with 16-wide tiles; X, Y: its
// operands (x per component, y as (own+next, own) per party), xcols: x holds the columns and y the nodes
struct CountArgs { LimbSet A, B; LimbTri X; LimbSet Y; int xcols; u64 nblk; u32 nh, ncol; u64 bcol0; u32 zcol0; u64 *Zacc; u32 nchunk, nrowgrp, nwide, rt, chunkblk, ncoltiles;   // ncoltiles: column tiles of 32*NB in this launch; nwide: slots per chunk that they take
                   u32 nns; u64 nbcol0; u32 nzcol0; };

// A remainder of at most 16 columns (the class totals), or all columns of few nodes: 16 rows of x per wavefront with
// v_mfma_i32_16x16x64_i8 (lane l holds row or column l%16 and the 16 samples
// 16*(l/16).. of a pair of sample blocks; result C[4*(l/16)+v][l%16]), for ALL THREE
// parties at once.  With so few columns the products are limited by the rate at which L
// arrives, so every component x_j is fetched once and multiplied by one tile that
// holds both operands it meets in the three-term products,
//   columns 0-7:  up to 8 rows of (y_j + y_{j+1})   ->  Z_j     (x_j is party j's own part)
//   columns 8-15: the same rows of y_{j-1}          ->  Z_{j-1} (and party j-1's next part)
// (each party's sums still come from the two components that party holds); rows y0 .. y1-1 of y in
// passes of 8.  It runs inside the launch of the wide groups, as one more column group of each
// sample chunk.  nx: rows of x that exist from x0 on.
// XCOLS (a.xcols): x holds the columns; the operands change places, so that lane l holds sums of column l%16 and the 16
// columns of a node are added to consecutive words.  The adds of all chunks to a line wait for each other: with a lane's four sums
// in four columns an instruction touched each line with four words only, 0.25 us a chunk, now 0.1 (50,000 samples
// x 34 columns, 1 to 8 nodes: 65-72 us, now 31-32; 500 x 4,002, 8 nodes: 87, now 34).
template <bool XCOLS>
__device__ __forceinline__ void count_narrow(const CountArgs &a, u64 x0, u32 nx, u64 y0, u64 y1, u64 ib0, u64 ib1, int lane)
{
    const u32 lr = lane & 15, kq = lane >> 4, half = (kq & 1) * 16;
    for (u64 yb = y0; yb < y1; yb += 8) {
        const u32 nc = y1 - yb < 8 ? (u32)(y1 - yb) : 8;
        const bool bcol = (lr & 7) < nc;                 // this lane's column of the tile exists
        const u64 brow = yb + (lr & 7);
        v4i acc[3][8];
#pragma unroll
        for (int j = 0; j < 3; j++)
#pragma unroll
            for (int u = 0; u < 8; u++) acc[j][u] = v4i{ 0, 0, 0, 0 };
        v4i A[3][8], B[3][8];
        // the lane's sample block of a pair; the second block of an odd tail does not belong
        // to this chunk: its lanes load the first block again and multiply zeros
#define CN_LOAD_A(J, IB)                                                                      \
        {                                                                                     \
            const u64 ibl = (IB) + (kq >> 1) >= ib1 ? (IB) : (IB) + (kq >> 1);                \
            _Pragma("unroll") for (int sl = 0; sl < 8; sl++)                                  \
                A[J][sl] = *(const v4i *)(a.X.m[J].base + limb_addr(a.X.m[J], ibl, sl, x0 + lr) + half); \
        }
#define CN_LOAD_B(J, IB)                                                                      \
        {                                                                                     \
            const bool tail = (IB) + (kq >> 1) >= ib1;                                        \
            const u64 ibl = tail ? (IB) : (IB) + (kq >> 1);                                   \
            const LimbMat &Bs_ = a.Y.m[J][0], &Bo_ = a.Y.m[((J) + 2) % 3][1];                 \
            const LimbMat bb_ = { lr < 8 ? Bs_.base : Bo_.base, lr < 8 ? Bs_.rows : Bo_.rows };\
            _Pragma("unroll") for (int sl = 0; sl < 8; sl++) {                                \
                B[J][sl] = v4i{ 0, 0, 0, 0 };                                                 \
                if (!tail && bcol) B[J][sl] = *(const v4i *)(bb_.base + limb_addr(bb_, ibl, sl, brow) + half); \
            }                                                                                 \
        }
#define CN_MMA(J)                                                                             \
        _Pragma("unroll") for (int sl = 0; sl < 8; sl++)                                      \
            _Pragma("unroll") for (int t = 0; t < 8 - sl; t++)                                \
                acc[J][sl + t] = XCOLS ? __builtin_amdgcn_mfma_i32_16x16x64_i8(B[J][t], A[J][sl], acc[J][sl + t], 0, 0, 0) \
                                       : __builtin_amdgcn_mfma_i32_16x16x64_i8(A[J][sl], B[J][t], acc[J][sl + t], 0, 0, 0);
        // 16 loads between the first MFMAs of the stage, one by one (see k_count)
#define CN_SPREAD()                                                                           \
        _Pragma("unroll") for (int q_ = 0; q_ < 16; q_++) {                                   \
            __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);                                \
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                                \
        }                                                                                     \
        __builtin_amdgcn_sched_group_barrier(0x008, 20, 0);                                   \
        __builtin_amdgcn_sched_barrier(0);
        // One pair of sample blocks = three stages of 36 MFMAs, one per component.  While a stage
        // multiplies, L for the stage after the next and the columns for the next are fetched.
        CN_LOAD_A(0, ib0)
        CN_LOAD_A(1, ib0)
        CN_LOAD_B(0, ib0)
        for (u64 ib = ib0; ib < ib1; ib += 2) {
            // the loads for the pair after the last are issued all the same (they read the chunk's
            // last pair again and are not used): the number of loads in flight stays fixed
            const u64 ibn = ib + 2 < ib1 ? ib + 2 : ib;
            __builtin_amdgcn_sched_barrier(0);
            CN_LOAD_A(2, ib)  CN_LOAD_B(1, ib)  CN_MMA(0) CN_SPREAD()
            CN_LOAD_A(0, ibn) CN_LOAD_B(2, ib)  CN_MMA(1) CN_SPREAD()
            CN_LOAD_A(1, ibn) CN_LOAD_B(0, ibn) CN_MMA(2) CN_SPREAD()
        }
#undef CN_LOAD_A
#undef CN_LOAD_B
#undef CN_MMA
#undef CN_SPREAD
#pragma unroll
        for (int j = 0; j < 3; j++) {
#pragma unroll
            for (int v = 0; v < 4; v++) {
                // row of x and of the 16 of y that this sum belongs to
                const u32 xr = XCOLS ? lr : 4 * kq + v, yr = XCOLS ? 4 * kq + v : lr;
                const int pz = yr < 8 ? j : (j + 2) % 3;     // the party whose sum it is
                const u64 x = x0 + xr, y = yb + (yr & 7), r = XCOLS ? y : x, c = a.nzcol0 + (XCOLS ? x : y) - a.nbcol0;
                u64 z = 0;
#pragma unroll
                for (int u = 0; u < 8; u++) z += (u64)(long long)acc[j][u][v] << (8 * u);
                if (xr < nx && (yr & 7) < nc) atomicAdd((unsigned long long *)&a.Zacc[((u64)pz * a.nh + r) * a.ncol + c], (unsigned long long)z);
            }
        }
    }
}

// Workgroup = 4 wavefronts, each 32 rows x (32*NB) columns of one party: rt row tiles (4, 2 or 1, by the nodes)
// x 4/rt tiles of columns and parties; NB = 2 for full groups of 64 columns, NB = 1 for a remainder of at
// most 32.  Bound: with 128 rows and more the matrix cores (busy 0.73 at the 1.4 GHz that their power leaves:
// 2.1 POP/s for 128 x 260 columns of 10^6 samples, a large int8 product of the vendor library reaches 2.0); with
// few rows the rate at which the operands arrive (about 24 KB per wavefront and product, rows below 32 are
// padding).  The operands of the next product are in flight while the current one is multiplied.
template <int NB>
__global__ __launch_bounds__(256) void k_count(CountArgs a)
{
    const int lane = threadIdx.x & 63;
    const u32 wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // Workgroups go round-robin to the 8 XCDs, each with its own L2.  The column groups of
    // one sample chunk, of all three parties, read the same rows of the three components of
    // L, so they are given consecutive slots of the same XCD: id = slot*8 + xcd; per chunk
    // nwide wide slots and nns narrow ones.  The column tiles of the three parties are dealt out to the
    // wavefronts of the wide slots one after the other (with a slot per party and group of tiles, nine
    // tiles of 64 columns left a quarter of the wavefronts without work), the three parties of a tile
    // side by side where x holds the columns (each component of a tile is read by two of them), party
    // by party otherwise.
    const u32 per = a.nwide + a.nns, id = blockIdx.x, xcd = id & 7, slot = id >> 3;
    const u32 sl = slot % per, chunk = (slot / per) * 8 + xcd;
    if (chunk >= a.nchunk) return;                            // whole workgroup, no barrier in this kernel
    const u64 ib0 = (u64)chunk * a.chunkblk;
    const u64 ib1 = ib0 + a.chunkblk < a.nblk ? ib0 + a.chunkblk : a.nblk;
    const u32 rg = blockIdx.z;
    if (sl >= a.nwide) {
        // a narrow slot of this chunk: its workgroups of 4 wavefronts share out the nodes, 16 rows of x
        // (each tile for all three parties) or, where x holds the columns, 8 rows of y and 16 columns per wavefront, the
        // wavefronts of the same columns side by side
        const u64 wv = ((u64)(sl - a.nwide) * a.nrowgrp + rg) * 4 + wave;
        const u32 nreal = a.ncol - a.nzcol0;
        if (a.xcols) {
            const u32 ny = (a.nh + 7) / 8;
            const u64 y0 = wv % ny * 8, c0 = wv / ny * 16;
            if (c0 < nreal) count_narrow<true>(a, a.nbcol0 + c0, nreal - c0 < 16 ? (u32)(nreal - c0) : 16, y0, y0 + 8 < a.nh ? y0 + 8 : a.nh, ib0, ib1, lane);
        } else if (wv * 16 < a.nh) {
            const u64 left = a.nh - wv * 16;
            count_narrow<false>(a, wv * 16, left < 16 ? (u32)left : 16, a.nbcol0, a.nbcol0 + nreal, ib0, ib1, lane);
        }
        return;
    }
    const u32 wr = wave % a.rt, task = sl * (4 / a.rt) + wave / a.rt;   // this wavefront's row tile, party and column tile
    if (task >= 3 * a.ncoltiles) return;                      // whole wavefront
    const bool beside = a.xcols && a.rt < 4;                  // four row tiles: the nodes' operands are the larger part
    const int p = beside ? task % 3 : task / a.ncoltiles;
    const u64 r0 = ((u64)rg * a.rt + wr) * 32;
    if (r0 >= a.nh) return;                                   // whole wavefront
    const LimbMat LA0 = p == 0 ? a.A.m[0][0] : (p == 1 ? a.A.m[1][0] : a.A.m[2][0]);
    const LimbMat LA1 = p == 0 ? a.A.m[0][1] : (p == 1 ? a.A.m[1][1] : a.A.m[2][1]);
    const LimbMat LB0 = p == 0 ? a.B.m[0][0] : (p == 1 ? a.B.m[1][0] : a.B.m[2][0]);
    const LimbMat LB1 = p == 0 ? a.B.m[0][1] : (p == 1 ? a.B.m[1][1] : a.B.m[2][1]);
    const u64 ctile = beside ? task / 3 : task % a.ncoltiles;    // column tile of 32*NB
    const u64 c0 = a.bcol0 + ctile * (32 * NB);
    const u32 lr = lane & 31;
    v16i acc[8][NB];
#pragma unroll
    for (int u = 0; u < 8; u++)
#pragma unroll
        for (int nb = 0; nb < NB; nb++)
#pragma unroll
            for (int v = 0; v < 16; v++) acc[u][nb][v] = 0;
    // addresses = wave-uniform base (scalar registers) + a 32-bit lane offset
    const u32 offA = (u32)((r0 + lr) * 32 + (lane >> 5) * 16), offB = (u32)(lr * 32 + (lane >> 5) * 16);
    v4i av0[8], bv0[NB][8], av1[8], bv1[NB][8];
#define CT_LOAD(AV, BV, LA, LB, IB)                                                           \
    _Pragma("unroll") for (int s = 0; s < 8; s++) {                                           \
        AV[s] = *(const v4i *)(LA.base + limb_addr(LA, IB, s, 0) + offA);                     \
        _Pragma("unroll") for (int nb = 0; nb < NB; nb++)                                     \
            BV[nb][s] = *(const v4i *)(LB.base + limb_addr(LB, IB, s, c0 + nb * 32) + offB);  \
    }
    // limb s of the left operand against limbs 0..7-s of the right one: successive MFMAs
    // go to different accumulators (level s+t), none waits for the one before it
#define CT_MMA(AV, BV)                                                                        \
    _Pragma("unroll") for (int s = 0; s < 8; s++)                                             \
        _Pragma("unroll") for (int t = 0; t < 8 - s; t++)                                     \
            _Pragma("unroll") for (int nb = 0; nb < NB; nb++)                                 \
                acc[s + t][nb] = __builtin_amdgcn_mfma_i32_32x32x32_i8(AV[s], BV[nb][t], acc[s + t][nb], 0, 0, 0);
    // The loads of the next product are issued one by one between the first MFMAs of this
    // product (a burst of 8*(1+NB) loads at once fills the L1 cache's queue of outstanding
    // misses and the matrix cores wait for it to drain); without the scheduling groups
    // the compiler would sink the loads to their uses to save registers.
#define CT_SPREAD()                                                                           \
    _Pragma("unroll") for (int q = 0; q < 8 * (1 + NB); q++) {                                \
        __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);                                    \
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                                    \
    }                                                                                         \
    __builtin_amdgcn_sched_group_barrier(0x008, 36 * NB - 8 * (1 + NB), 0);
    CT_LOAD(av0, bv0, LA0, LB0, ib0)
    for (u64 ib = ib0; ib < ib1; ib++) {
        __builtin_amdgcn_sched_barrier(0);
        CT_LOAD(av1, bv1, LA1, LB1, ib)
        CT_MMA(av0, bv0)
        CT_SPREAD()
        __builtin_amdgcn_sched_barrier(0);
        // always issued (the last one re-reads the chunk's last block and is not used): with a
        // fixed number of loads in flight the wait before the next product leaves them pending
        CT_LOAD(av0, bv0, LA0, LB0, (ib + 1 < ib1 ? ib + 1 : ib))
        CT_MMA(av1, bv1)
        CT_SPREAD()
        __builtin_amdgcn_sched_barrier(0);
    }
#undef CT_SPREAD
#undef CT_LOAD
#undef CT_MMA
    u64 *Z = a.Zacc + (u64)p * a.nh * a.ncol;
#pragma unroll
    for (int nb = 0; nb < NB; nb++)
#pragma unroll
        for (int v = 0; v < 16; v++) {
            const u64 r = r0 + 8 * (v / 4) + 4 * (lane >> 5) + (v & 3);
            const u64 c = a.zcol0 + ctile * (32 * NB) + nb * 32 + lr;
            u64 z = 0;
#pragma unroll
            for (int u = 0; u < 8; u++) z += (u64)(long long)acc[u][nb][v] << (8 * u);
            if (r < a.nh && c < a.ncol) atomicAdd((unsigned long long *)&Z[r * a.ncol + c], (unsigned long long)z);
        }
}

// add the zero sharing, reshare, accumulate into the node statistics
struct CountFinArgs { KCommon c; u64 *Zacc; P6 C; u64 n; u32 ncol, CW; u64 colbase; };
__global__ __launch_bounds__(64) void k_count_fin(CountFinArgs a)
{
    GT_EL_SHARED(1, PRF_ALONE)
    GT_FOR_EL(a.n) {
        const u64 e0 = tile_ * GT_EL, o = e0 + W.t, idx = (o / a.ncol) * a.CW + a.colbase + o % a.ncol;
        const bool act = W.t < GT_EL && o < a.n;
        const u32 s0[1] = { 0 };
        Sh z, old = { 0, 0 };
        u64 part = 0;
        if (act) { part = a.Zacc[(u64)p * a.n + o]; old = ld(a.C, p, idx); }
        T.deal(W, a.c.op, e0, s0, 0);
        if (act) a.Zacc[(u64)p * a.n + o] = 0;         // zero again for the next contraction
        z.o = part + T.za(W, 0, (u32)(e0 & 7) + W.t);
        z.n = W.reshare1(z.o, act ? 64u : 0u);
        if (act && W.real) st(a.C, p, idx, old + z);
        W.drain();
    }
    W.flush(a.c.wire);
}

// counter-array layout of Sec. V-B for export: per node (1+K) x 2d, local linear ops
__global__ __launch_bounds__(256) void k_c_paper(P6 C, P6 out, u32 nh, u32 d, u32 K, u32 CW)
{
    const u64 per = (u64)(1 + K) * 2 * d, n = (u64)nh * per;
    for (u64 t = (u64)blockIdx.x * blockDim.x + threadIdx.x; t < n; t += (u64)gridDim.x * blockDim.x) {
        const u64 r = t / per, q = t % per, row = q / (2 * d), col = q % (2 * d), k = col / 2, v = col & 1;
        for (int j = 0; j < 3; j++)
            for (int pl = 0; pl < 2; pl++) {
                const u64 *src = pl ? C.n[j] : C.o[j];
                u64 val = 0;
                for (u32 cl = (row ? row - 1 : 0); cl < (row ? row : K); cl++) {
                    const u64 n1 = src[r * CW + k * K + cl], tot = src[r * CW + (u64)d * K + cl];
                    val += v ? n1 : tot - n1;
                }
                (pl ? out.n[j] : out.o[j])[t] = val;
            }
    }
}
