// Device-side toolkit: PRF, per-party share arithmetic, message exchange and the
// per-element protocol steps (Sec. II-B and Sec. V-A of the GTree paper), for gfx950.
//
// Execution models.  Wavefront model (WWire, ElTile, further down): the three parties of an
// element sit in three lanes of one wavefront; equality grids, inference and the per-node
// protocols run like this.  Workgroup model (products, one-time products, partition by
// products, the protocols as printed): a workgroup is 3 wavefronts of 64 lanes, wavefront p IS
// party p (threadIdx.y = p), lane l of each works on the same element(s).  Either way a
// party's lane holds its own two components, a protocol message is a store into a message
// region in LDS that the receiving party's lane loads (after a workgroup barrier in the second
// model), and a party's lanes use no component that the party does not hold and nothing of another
// party's but the words sent to it.  Where a component is stored once for both of its holders (a
// training's data and tiles, the values of an inference) or read once for both (products' factors,
// instances, a training's input), party p takes its next component from the place of party p + 1's own,
// which equals its own copy: less to read where the three parties share a GPU's memory, and only there.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "gt_shape.hpp"

#define GT_LANES 64
#define GT_KEY_DEALER 3
#define GT_KEY_OWNER 4

// ---------------------------------------------------------------------------------
// ChaCha block function, 8 rounds, as a counter-based PRF.  State words 12..15 are
// (block lo, block hi, op, stream); output word w (64 bit) is the little-endian pair
// (2w, 2w+1).  A key is wave-uniform and in scalar registers (load_key) where a wavefront is a party, per lane and
// in vector registers where its lanes take different roles (load_lane_key, ElTile, k_infer).
struct Key { u32 k[8]; };

__device__ __forceinline__ u32 rotl32(u32 x, int r) { return __builtin_rotateleft32(x, r); }

#ifndef GT_PRF_ROUNDS
#define GT_PRF_ROUNDS 8          // ChaCha rounds of the PRF (the CPU check uses the same number)
#endif
// Issue.  A SIMD issues a vector instruction every 4 cycles, but one of each of two wavefronts together when
// both are additions, subtractions, moves or plain logic of up to three inputs (vector registers or
// immediates); a shift, rotation, permute, multiply, carry or scalar operand goes alone.  Two thirds of a block are
// of the first kind, yet with the wavefronts served oldest first next to none of them pair: the older one goes
// ahead into its additions while the younger waits at a rotation, and so on.  So the rotations of a step are issued at
// the highest wavefront priority, additions and exclusive ors at the lowest, the rest of a kernel (mostly of the
// second kind) in between: whoever stands at a rotation goes first, and the two wavefronts meet again at the additions.
// Blocks alone, cycles per instruction: with two wavefronts per SIMD 4.53 -> 2.60, with four 4.08 -> 2.62, with eight 4.09 -> 2.41.
// Array access 200,003 x 100 269 -> 210 us, 100,003 quotients 109 -> 75 us; the same priority for additions and the rest: 225 and 87.
// PRF_ALONE: none of this, where a SIMD has one wavefront as a rule (4.91 -> 5.00 cycles).  PRF_PAIR_LOOP: in loops that call this
// with one key, operation and stream three of the first round's quarter rounds are constants and leave the loop; the first
// round goes without priorities then (10^6 instances of depth 10: 28.9 ms, 30.9 with them; the quotients 77 us without, 75 with).
enum { PRF_ALONE = 0, PRF_PAIR = 1, PRF_PAIR_LOOP = 2 };
#define GT_PRIO_ADD 0
#define GT_PRIO_REST 1
#define GT_PRIO_ROT 3
// sets the priority behind the computation of the four words
template <bool PAIR, int PRIO>
__device__ __forceinline__ void prf_prio(u32 a, u32 b, u32 c, u32 d)
{
    if (PAIR) {
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_setprio %4" :: "v"(a), "v"(b), "v"(c), "v"(d), "n"(PRIO));
        __builtin_amdgcn_sched_barrier(0);
    }
}
// the step a += b, d ^= a, d <<<= r of four quarter rounds
template <bool PAIR, int AFTER = GT_PRIO_ADD>
__device__ __forceinline__ void prf_step(u32 &a0, u32 &a1, u32 &a2, u32 &a3, u32 b0, u32 b1, u32 b2, u32 b3, u32 &d0, u32 &d1, u32 &d2, u32 &d3, int r)
{
    a0 += b0; a1 += b1; a2 += b2; a3 += b3;
    d0 ^= a0; d1 ^= a1; d2 ^= a2; d3 ^= a3;
    prf_prio<PAIR, GT_PRIO_ROT>(d0, d1, d2, d3);
    d0 = rotl32(d0, r); d1 = rotl32(d1, r); d2 = rotl32(d2, r); d3 = rotl32(d3, r);
    prf_prio<PAIR, AFTER>(d0, d1, d2, d3);
}
// four quarter rounds, on (a0, b0, c0, d0) and so on
template <bool PAIR, int AFTER = GT_PRIO_ADD>
__device__ __forceinline__ void prf_quarters(u32 &a0, u32 &a1, u32 &a2, u32 &a3, u32 &b0, u32 &b1, u32 &b2, u32 &b3,
                                             u32 &c0, u32 &c1, u32 &c2, u32 &c3, u32 &d0, u32 &d1, u32 &d2, u32 &d3)
{
    prf_step<PAIR>(a0, a1, a2, a3, b0, b1, b2, b3, d0, d1, d2, d3, 16);
    prf_step<PAIR>(c0, c1, c2, c3, d0, d1, d2, d3, b0, b1, b2, b3, 12);
    prf_step<PAIR>(a0, a1, a2, a3, b0, b1, b2, b3, d0, d1, d2, d3, 8);
    prf_step<PAIR, AFTER>(c0, c1, c2, c3, d0, d1, d2, d3, b0, b1, b2, b3, 7);
}
template <int ISSUE = PRF_ALONE>
__device__ __forceinline__ void chacha8(const Key &key, u64 blk, u32 op, u32 stream, u64 (&out)[8])
{
    constexpr bool PAIR = ISSUE != PRF_ALONE;
    const u32 i0 = 0x61707865u, i1 = 0x3320646eu, i2 = 0x79622d32u, i3 = 0x6b206574u;
    const u32 c12 = (u32)blk, c13 = (u32)(blk >> 32);
    u32 x0 = i0, x1 = i1, x2 = i2, x3 = i3;
    u32 x4 = key.k[0], x5 = key.k[1], x6 = key.k[2], x7 = key.k[3];
    u32 x8 = key.k[4], x9 = key.k[5], x10 = key.k[6], x11 = key.k[7];
    u32 x12 = c12, x13 = c13, x14 = op, x15 = stream;
    prf_quarters<ISSUE == PRF_PAIR>(x0, x1, x2, x3, x4, x5, x6, x7, x8, x9, x10, x11, x12, x13, x14, x15);
#pragma unroll
    for (int r = 1; r < GT_PRF_ROUNDS - 1; r += 2) {
        prf_quarters<PAIR>(x0, x1, x2, x3, x5, x6, x7, x4, x10, x11, x8, x9, x15, x12, x13, x14);
        prf_quarters<PAIR>(x0, x1, x2, x3, x4, x5, x6, x7, x8, x9, x10, x11, x12, x13, x14, x15);
    }
    prf_quarters<PAIR, GT_PRIO_REST>(x0, x1, x2, x3, x5, x6, x7, x4, x10, x11, x8, x9, x15, x12, x13, x14);
    x0 += i0; x1 += i1; x2 += i2; x3 += i3;
    x4 += key.k[0]; x5 += key.k[1]; x6 += key.k[2]; x7 += key.k[3];
    x8 += key.k[4]; x9 += key.k[5]; x10 += key.k[6]; x11 += key.k[7];
    x12 += c12; x13 += c13; x14 += op; x15 += stream;
    out[0] = (u64)x0 | ((u64)x1 << 32);   out[1] = (u64)x2 | ((u64)x3 << 32);
    out[2] = (u64)x4 | ((u64)x5 << 32);   out[3] = (u64)x6 | ((u64)x7 << 32);
    out[4] = (u64)x8 | ((u64)x9 << 32);   out[5] = (u64)x10 | ((u64)x11 << 32);
    out[6] = (u64)x12 | ((u64)x13 << 32); out[7] = (u64)x14 | ((u64)x15 << 32);
}

__device__ __forceinline__ Key load_key(const u32 *keys, int idx)
{
    Key k;
#pragma unroll
    for (int i = 0; i < 8; i++) k.k[i] = __builtin_amdgcn_readfirstlane(keys[idx * 8 + i]);
    return k;
}

// The keys one party may use: its two pairwise keys (Sec. III) and, in this
// simulation, the dealer key from which the offline material is derived.
// scr: this wavefront's 8 x 64 words of LDS for handing PRF words round its lanes
// (kernels with one element per lane, see prf_tile), else null.
struct PartyKeys { Key own, nxt, dlr; u64 *scr; };
#define GT_PRF_SCRATCH_WORDS (8 * GT_LANES)

__device__ __forceinline__ PartyKeys load_party_keys(const u32 *keys, int p, u64 *scr = nullptr)
{
    PartyKeys K;
    K.own = load_key(keys, p);
    K.nxt = load_key(keys, p == 2 ? 0 : p + 1);
    K.dlr = load_key(keys, GT_KEY_DEALER);
    K.scr = scr;
    return K;
}

// Words of NS streams under the own and the next key for a tile of 64 consecutive
// elements, element 64*tile + lane in lane `lane` (every kernel with one element per
// lane indexes that way, and all 64 lanes call together).  A block of the PRF holds
// the words of 8 consecutive elements, so the tile needs 8 blocks per key and stream:
// lane l < 16*NS evaluates block l%8 of stream (l/16), own key if (l/8) is even, next key
// otherwise, and leaves its 8 words in the wavefront's scratch; then every lane picks
// its own.  One pass of the block function instead of 2*NS.  LDS operations of one
// wavefront complete in order, so no hardware barrier is needed; the wavefront-scope
// fences keep the compiler from moving the loads of other lanes' words across the stores.
template <int NS>
__device__ __forceinline__ void prf_tile(const PartyKeys &K, u32 op, const u32 (&st)[NS], u64 e, u64 (&wo)[NS], u64 (&wn)[NS])
{
    static_assert(NS >= 1 && NS <= 4, "at most 8 key/stream pairs per pass");
    const u32 lane = threadIdx.x, c = lane >> 3;
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");      // the previous call's loads come first
    __builtin_amdgcn_wave_barrier();
    if (c < 2 * NS) {
        // selections by masks: plain ALU work on the scalar key words
        const u32 mk = 0u - (c & 1);
        Key kv;
#pragma unroll
        for (int i = 0; i < 8; i++) kv.k[i] = K.own.k[i] ^ ((K.own.k[i] ^ K.nxt.k[i]) & mk);
        u32 stream = 0;
#pragma unroll
        for (int q = 0; q < NS; q++) stream |= st[q] & (0u - (u32)((c >> 1) == (u32)q));
        u64 blk[8];
        chacha8(kv, (e >> 6) * 8 + (lane & 7), op, stream, blk);
#pragma unroll
        for (int i = 0; i < 8; i++) K.scr[c * GT_LANES + (lane & 7) * 8 + i] = blk[i];
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int q = 0; q < NS; q++) { wo[q] = K.scr[(2 * q) * GT_LANES + lane]; wn[q] = K.scr[(2 * q + 1) * GT_LANES + lane]; }
}

// party p's component of the zero sharing of element e: arithmetic / Boolean
__device__ __forceinline__ u64 zero_a(const PartyKeys &K, u32 op, u32 stream, u64 e)
{
    const u32 st[1] = { stream }; u64 wo[1], wn[1];
    prf_tile<1>(K, op, st, e, wo, wn);
    return wo[0] - wn[0];
}
__device__ __forceinline__ u64 zero_b(const PartyKeys &K, u32 op, u32 stream, u64 e)
{
    const u32 st[1] = { stream }; u64 wo[1], wn[1];
    prf_tile<1>(K, op, st, e, wo, wn);
    return wo[0] ^ wn[0];
}
// two streams in one pass
__device__ __forceinline__ void zero_b2(const PartyKeys &K, u32 op, u32 s0, u32 s1, u64 e, u64 &z0, u64 &z1)
{
    const u32 st[2] = { s0, s1 }; u64 wo[2], wn[2];
    prf_tile<2>(K, op, st, e, wo, wn);
    z0 = wo[0] ^ wn[0]; z1 = wo[1] ^ wn[1];
}

// ---------------------------------------------------------------------------------
// A party's view of one shared element: components p (own) and p+1 (next).
struct Sh { u64 o, n; };

// kernel-argument view of a shared vector: six planes
struct P6 { u64 *o[3]; u64 *n[3]; };

__device__ __forceinline__ u64 *own_of(const P6 &a, int p) { return p == 0 ? a.o[0] : (p == 1 ? a.o[1] : a.o[2]); }
__device__ __forceinline__ u64 *nxt_of(const P6 &a, int p) { return p == 0 ? a.n[0] : (p == 1 ? a.n[1] : a.n[2]); }
__device__ __forceinline__ Sh ld(const P6 &a, int p, size_t e) { Sh v; v.o = own_of(a, p)[e]; v.n = nxt_of(a, p)[e]; return v; }
__device__ __forceinline__ void st(const P6 &a, int p, size_t e, Sh v) { own_of(a, p)[e] = v.o; nxt_of(a, p)[e] = v.n; }

// public constant c as the sharing (c, 0, 0): component 1 is party 0's own and party 2's next
__device__ __forceinline__ Sh pub(int p, u64 c) { Sh v; v.o = p == 0 ? c : 0; v.n = p == 2 ? c : 0; return v; }
__device__ __forceinline__ Sh operator+(Sh a, Sh b) { Sh v; v.o = a.o + b.o; v.n = a.n + b.n; return v; }
__device__ __forceinline__ Sh operator-(Sh a, Sh b) { Sh v; v.o = a.o - b.o; v.n = a.n - b.n; return v; }
__device__ __forceinline__ Sh operator^(Sh a, Sh b) { Sh v; v.o = a.o ^ b.o; v.n = a.n ^ b.n; return v; }
__device__ __forceinline__ Sh scale(Sh a, u64 c) { Sh v; v.o = a.o * c; v.n = a.n * c; return v; }

// party-local part of a product: z_p = x_p y_p + x_{p+1} y_p + x_p y_{p+1}
__device__ __forceinline__ u64 prod3(Sh x, Sh y) { return x.o * (y.o + y.n) + x.n * y.o; }
// three-input logic, one instruction: T is the value of the expression on a = 0xf0, b = 0xcc, c = 0xaa
template <u32 T> __device__ __forceinline__ u32 logic3(u32 a, u32 b, u32 c) { return __builtin_amdgcn_bitop3_b32(a, b, c, T); }
// x_o y_o + x_o y_n + x_n y_o over bits (the three-term product), two instructions
__device__ __forceinline__ u32 and3l(u32 ao, u32 an, u32 bo, u32 bn) { return logic3<0x6a>(an, bo, logic3<0x60>(ao, bo, bn)); }
__device__ __forceinline__ u32 xor3l(u32 a, u32 b, u32 c) { return logic3<0x96>(a, b, c); }
__device__ __forceinline__ u64 and3(Sh x, Sh y)
{
    return (u64)and3l((u32)x.o, (u32)x.n, (u32)y.o, (u32)y.n)
         | ((u64)and3l((u32)(x.o >> 32), (u32)(x.n >> 32), (u32)(y.o >> 32), (u32)(y.n >> 32)) << 32);
}

// The party of this wavefront.  All 64 lanes of a wavefront share threadIdx.y (the
// workgroup is 64 x 3), so the value is read into a scalar register: selections and
// branches on the party then cost no vector instructions.
__device__ __forceinline__ int party_of_wave() { return __builtin_amdgcn_readfirstlane((int)threadIdx.y); }

// ---------------------------------------------------------------------------------
// Message exchange inside the workgroup.  `reshare`: every party sends to its
// predecessor (after a product, so that the receiver then holds (z_p, z_{p+1}));
// `open`: every party sends to its successor (it hands over its first component).
// The message region is GT_LWIRE_WORDS words of LDS that the workgroup owns: two
// alternating slots for messages of up to four words per lane, so that one barrier per
// message suffices (a slot is rewritten only after the barrier of the message that
// followed it).
#define GT_WIRE_SLOTS 64
#define GT_LWIRE_SLOT (3 * 4 * GT_LANES)
#define GT_LWIRE_WORDS (2 * GT_LWIRE_SLOT)
// Every send states how many payload bits the lane's message carries (0 for a lane whose
// element does not exist); the lane adds them up per direction, the sums are collected
// per party in six words of LDS (drain) and handed to the context's counters when the
// kernel ends (flush), so that the bytes reported for a call are counted where the
// messages are stored, not derived from the sizes on the host.  Party p's wavefront is the
// only one that touches words 2p and 2p+1 of the LDS counters, and the LDS operations of
// one wavefront complete in order, so the counting needs no barrier.
struct LWire {
    u64 *base, *cnt;
    int slot, p, lane;
    u32 nopen, nresh;            // payload bits this lane has sent to its successor / predecessor since the last drain
    __device__ __forceinline__ void init(u64 *lds, u64 *s_cnt)
    {
        base = lds; cnt = s_cnt; slot = 0; p = party_of_wave(); lane = threadIdx.x; nopen = 0; nresh = 0;
        if (lane < 2) cnt[2 * p + lane] = 0;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
    template <int NW>
    __device__ __forceinline__ void exchange(const u64 (&snd)[NW], u64 (&rcv)[NW], int from)
    {
        static_assert(NW <= 4, "message too wide");
        u64 *buf = base + slot * GT_LWIRE_SLOT;
        slot ^= 1;
#pragma unroll
        for (int j = 0; j < NW; j++) buf[(p * 4 + j) * GT_LANES + lane] = snd[j];
        __syncthreads();
#pragma unroll
        for (int j = 0; j < NW; j++) rcv[j] = buf[(from * 4 + j) * GT_LANES + lane];
    }
    template <int NW>
    __device__ __forceinline__ void reshare(const u64 (&snd)[NW], u64 (&rcv)[NW], u32 bits) { nresh += bits; exchange<NW>(snd, rcv, p == 2 ? 0 : p + 1); }
    template <int NW>
    __device__ __forceinline__ void open(const u64 (&snd)[NW], u64 (&rcv)[NW], u32 bits) { nopen += bits; exchange<NW>(snd, rcv, p == 0 ? 2 : p - 1); }
    __device__ __forceinline__ u64 reshare1(u64 v, u32 bits) { u64 s[1] = { v }, r[1]; reshare<1>(s, r, bits); return r[0]; }
    __device__ __forceinline__ u64 open1(u64 v, u32 bits) { u64 s[1] = { v }, r[1]; open<1>(s, r, bits); return r[0]; }
    // move the lane's sums into the party's LDS counters (long loops call it once per work
    // item, before the 32-bit sums could overflow)
    __device__ __forceinline__ void drain()
    {
        if (nopen) atomicAdd((unsigned long long *)&cnt[2 * p], (unsigned long long)nopen);
        if (nresh) atomicAdd((unsigned long long *)&cnt[2 * p + 1], (unsigned long long)nresh);
        nopen = 0; nresh = 0;
    }
    // end of the kernel: add the party's sums to the context's counters, g[6*slot + 2p] (bits
    // sent to the successor) and g[6*slot + 2p+1] (to the predecessor); the workgroups of a
    // launch spread over GT_WIRE_SLOTS slots so that their atomic adds do not queue up on one
    // address (the host adds the slots up).  Every lane calls it once.
    __device__ __forceinline__ void flush(u64 *g)
    {
        drain();
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        if (lane < 2) {
            const u64 v = cnt[2 * p + lane];
            const u32 slot = (blockIdx.x + blockIdx.y) & (GT_WIRE_SLOTS - 1);
            if (v) atomicAdd((unsigned long long *)&g[6 * slot + 2 * p + lane], (unsigned long long)v);
        }
    }
};
typedef LWire Wire;

// ---------------------------------------------------------------------------------
// Offline material of one element, party p's components (dealer stream 0, block e).
struct Dealer { Sh rA, rho, bA; u32 bBo, bBn; };

__device__ __forceinline__ Dealer dealer_from_block(const u64 (&D)[8], int p)
{
    const u64 r = D[0], beta = D[5] & 1;
    const u64 rA2 = r - D[1] - D[2], rho2 = r ^ D[3] ^ D[4], bA2 = beta - D[6] - D[7];
    const u32 b0 = (u32)(D[5] >> 1) & 1, b1 = (u32)(D[5] >> 2) & 1, b2 = ((u32)beta ^ b0 ^ b1) & 1;
    Dealer d;
    d.rA.o = p == 0 ? D[1] : (p == 1 ? D[2] : rA2);   d.rA.n = p == 0 ? D[2] : (p == 1 ? rA2 : D[1]);
    d.rho.o = p == 0 ? D[3] : (p == 1 ? D[4] : rho2); d.rho.n = p == 0 ? D[4] : (p == 1 ? rho2 : D[3]);
    d.bA.o = p == 0 ? D[6] : (p == 1 ? D[7] : bA2);   d.bA.n = p == 0 ? D[7] : (p == 1 ? bA2 : D[6]);
    d.bBo = p == 0 ? b0 : (p == 1 ? b1 : b2);         d.bBn = p == 0 ? b1 : (p == 1 ? b2 : b0);
    return d;
}

__device__ __forceinline__ Dealer dealer_of(const PartyKeys &K, int p, u32 op, u64 e)
{
    u64 D[8];
    chacha8(K.dlr, e, op, 0, D);
    return dealer_from_block(D, p);
}

// ---------------------------------------------------------------------------------
// Per-element protocols, one element per lane.  Every lane of the workgroup must
// call them together (they contain barriers); inactive lanes pass zeros.

// product with reshare: returns (z_p, z_{p+1})
template <class WireT>
__device__ __forceinline__ Sh mult_sh(WireT &W, Sh x, Sh y, u64 alpha, bool act)
{
    Sh z;
    z.o = prod3(x, y) + alpha;
    z.n = W.reshare1(z.o, act ? 64u : 0u);
    return z;
}

// Equality test [v == 0] -> Boolean bit sharing.  A receives the Boolean
// zero-sharing word of stream 1 (bits 0..62 used here, bit 63 free for a following AND).
template <class WireT>
__device__ __forceinline__ Sh eq_bit_mask(WireT &W, int p, Sh v, const Dealer &D, u64 A, bool act)
{
    Sh m = v + D.rA;
    const u64 c = m.o + m.n + W.open1(m.o, act ? 64u : 0u);
    Sh t = D.rho;
    if (p == 0) t.o ^= ~c;
    if (p == 2) t.n ^= ~c;
    u32 off = 0;
#pragma unroll
    for (int k = 0; k < 6; k++) {
        const u32 w = 32u >> k;
        const u64 mask = (w == 32) ? 0xffffffffull : ((1ull << w) - 1);
        Sh a, b;
        a.o = t.o & mask; a.n = t.n & mask;
        b.o = (t.o >> w) & mask; b.n = (t.n >> w) & mask;
        t.o = (and3(a, b) ^ (A >> off)) & mask;
        t.n = W.reshare1(t.o, act ? w : 0u);
        off += w;
    }
    return t;
}
__device__ __forceinline__ Sh eq_bit(Wire &W, const PartyKeys &K, int p, u32 op, u64 e, Sh v, const Dealer &D, u64 &A, bool act)
{
    A = zero_b(K, op, 1, e);
    return eq_bit_mask(W, p, v, D, A, act);
}

// one-bit AND with reshare; alpha is the mask bit
template <class WireT>
__device__ __forceinline__ Sh and_bit(WireT &W, Sh x, Sh y, u64 alpha, bool act)
{
    Sh z;
    z.o = (and3(x, y) ^ alpha) & 1;
    z.n = W.reshare1(z.o, act ? 1u : 0u);
    return z;
}

// Comparison [v >= 0] (v signed, |v| < 2^63) -> Boolean bit sharing.
// AG, AE: the lane's Boolean zero-sharing words of streams 1 and 2 (own xor next key).
template <class WireT>
__device__ __forceinline__ Sh ge_bit_masks(WireT &W, int p, Sh v, const Dealer &D, u64 AG, u64 AE, bool act)
{
    const u64 LOW63 = 0x7fffffffffffffffull, TOP = 0x8000000000000000ull;
    Sh m = v + D.rA;
    const u64 c = m.o + m.n + W.open1(m.o, act ? 64u : 0u);
    const u64 nc = ~c;
    Sh G, E;
    G.o = nc & D.rho.o & LOW63; G.n = nc & D.rho.n & LOW63;
    E.o = D.rho.o & LOW63;      E.n = D.rho.n & LOW63;
    if (p == 0) E.o = ((D.rho.o ^ nc) & LOW63) | TOP;
    if (p == 2) E.n = ((D.rho.n ^ nc) & LOW63) | TOP;
#pragma unroll
    for (int k = 0; k < 6; k++) {
        const int s = 1 << k;
        // positions that start a block of 2s bits
        const u64 sm = k == 0 ? 0x5555555555555555ull : k == 1 ? 0x1111111111111111ull
                     : k == 2 ? 0x0101010101010101ull : k == 3 ? 0x0001000100010001ull
                     : k == 4 ? 0x0000000100000001ull : 0x1ull;
        Sh Eh, Gh;
        Eh.o = E.o >> s; Eh.n = E.n >> s; Gh.o = G.o >> s; Gh.n = G.n >> s;
        const u64 zg = (and3(Eh, G) ^ (AG >> (s - 1))) & sm;
        if (k < 5) {
            const u64 ze = (and3(Eh, E) ^ (AE >> (s - 1))) & sm;
            u64 snd[2] = { zg, ze }, rcv[2];
            W.template reshare<2>(snd, rcv, act ? 2u * (32u >> k) : 0u);   // one bit per block start, G and E
            G.o = (Gh.o & sm) ^ zg; G.n = (Gh.n & sm) ^ rcv[0];
            E.o = ze; E.n = rcv[1];
        } else {
            const u64 r = W.reshare1(zg, act ? 1u : 0u);
            G.o = (Gh.o & sm) ^ zg; G.n = (Gh.n & sm) ^ r;
        }
    }
    Sh ge;
    ge.o = ((D.rho.o >> 63) ^ G.o) & 1;
    ge.n = ((D.rho.n >> 63) ^ G.n) & 1;
    if (p == 0) ge.o ^= (c >> 63) ^ 1;
    if (p == 2) ge.n ^= (c >> 63) ^ 1;
    return ge;
}

// the same with the mask words of element e taken from the wavefront's PRF tile
// (element 64*tile + lane in every lane)
__device__ __forceinline__ Sh ge_bit(Wire &W, const PartyKeys &K, int p, u32 op, u64 e, Sh v, const Dealer &D, bool act)
{
    u64 AG, AE;
    zero_b2(K, op, 1, 2, e, AG, AE);
    return ge_bit_masks(W, p, v, D, AG, AE, act);
}

// bit -> arithmetic: open f = s xor beta; s = beta if f = 0 else 1 - beta
// (bits: what the opened value is counted as - one bit, or a ring element of 64 bits where
// the protocol is run as the paper's cost formula prices it)
template <class WireT>
__device__ __forceinline__ Sh b2a(WireT &W, int p, Sh s, const Dealer &D, bool act, u32 bits = 1)
{
    const u64 fo = (s.o ^ D.bBo) & 1, fn = (s.n ^ D.bBn) & 1;
    const u64 f = (fo ^ fn ^ W.open1(fo, act ? bits : 0u)) & 1;
    Sh one = pub(p, 1), out;
    out.o = f ? one.o - D.bA.o : D.bA.o;
    out.n = f ? one.n - D.bA.n : D.bA.n;
    return out;
}

__device__ __forceinline__ Sh not_bit(int p, Sh b) { if (p == 0) b.o ^= 1; if (p == 2) b.n ^= 1; return b; }

// ---------------------------------------------------------------------------------
// Wavefront model: the three parties of one wavefront.  Lanes 0-20 are party 0, 21-41
// party 1, 42-62 party 2 (lane 63 repeats lane 62 and neither stores, counts nor adds), so
// lanes t, 21 + t and 42 + t work on the same elements, each on its party's two components
// and with its party's keys.  A message is a store into the wavefront's message region in LDS
// that the receiving party's lane loads; LDS operations of one wavefront complete in order,
// so no workgroup barrier is needed and the wavefronts of a compute unit run independently
// of each other.

// orders this wavefront's LDS accesses for the compiler (the hardware keeps their order)
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

#define GT_WMSG_QUADS (2 * GT_LANES)                 // message region of a wavefront: 8 dwords per lane
struct WWire {
    uint4 *buf;
    u64 *cnt;
    int p, pn;
    u32 m, t, nx, pv;            // this lane (63: as 62), its number in the party, the lanes of the next and the previous party
    bool real;
    u64 nopen, nresh;            // payload bits sent to the successor / predecessor since the last drain
    __device__ __forceinline__ void init(uint4 *region, u64 *s_cnt)
    {
        const u32 l = threadIdx.x & (GT_LANES - 1);
        real = l < 3 * GT_TP; m = real ? l : 3 * GT_TP - 1;
        p = m >= 2 * GT_TP ? 2 : (m >= GT_TP ? 1 : 0); pn = p == 2 ? 0 : p + 1;
        t = m - GT_TP * (u32)p;
        nx = p == 2 ? t : m + GT_TP; pv = p == 0 ? m + 2 * GT_TP : m - GT_TP;
        buf = region; cnt = s_cnt; nopen = 0; nresh = 0;
        if (cnt && l < 6) cnt[l] = 0;
        wave_sync();
    }
    __device__ __forceinline__ u32 lane_of(u32 e) const { return GT_TP * (u32)p + e; }     // the party's lane number e
    // store ND dwords, load those that lane `from` stored
    template <int ND>
    __device__ __forceinline__ void pass(const u32 (&s)[ND], u32 (&r)[ND], u32 from)
    {
        static_assert(ND == 1 || ND == 2 || (ND % 4 == 0 && ND <= 8), "message size");
        wave_sync();
        // small messages use the same 16-byte slots: one address register per direction for all sizes
        if (ND == 1) buf[m].x = s[0];
        else if (ND == 2) *(uint2 *)&buf[m] = make_uint2(s[0], s[ND > 1 ? 1 : 0]);
        else {
#pragma unroll
            for (int j = 0; j < ND / 4; j++) buf[j * GT_LANES + m] = make_uint4(s[4 * j], s[4 * j + 1], s[4 * j + 2], s[4 * j + 3]);
        }
        wave_sync();
        if (ND == 1) r[0] = buf[from].x;
        else if (ND == 2) { const uint2 v = *(const uint2 *)&buf[from]; r[0] = v.x; r[ND > 1 ? 1 : 0] = v.y; }
        else {
#pragma unroll
            for (int j = 0; j < ND / 4; j++) {
                const uint4 v = buf[j * GT_LANES + from];
                r[4 * j] = v.x; r[4 * j + 1] = v.y; r[4 * j + 2] = v.z; r[4 * j + 3] = v.w;
            }
        }
    }
    template <int NW>
    __device__ __forceinline__ void pass64(const u64 (&s)[NW], u64 (&r)[NW], u32 from)
    {
        constexpr int M = NW < 4 ? NW : 4;             // words at a time: the region's 8 dwords per lane
        static_assert(NW % M == 0, "message size");
#pragma unroll
        for (int h = 0; h < NW; h += M) {
            u32 a[2 * M], b[2 * M];
#pragma unroll
            for (int j = 0; j < M; j++) { a[2 * j] = (u32)s[h + j]; a[2 * j + 1] = (u32)(s[h + j] >> 32); }
            pass<2 * M>(a, b, from);
#pragma unroll
            for (int j = 0; j < M; j++) r[h + j] = (u64)b[2 * j] | ((u64)b[2 * j + 1] << 32);
        }
    }
    template <int ND> __device__ __forceinline__ void reshare(const u32 (&s)[ND], u32 (&r)[ND]) { pass<ND>(s, r, nx); }
    template <int NW> __device__ __forceinline__ void reshare64(const u64 (&s)[NW], u64 (&r)[NW]) { pass64<NW>(s, r, nx); }
    // the interface of LWire, for the per-element protocols
    template <int NW>
    __device__ __forceinline__ void reshare(const u64 (&s)[NW], u64 (&r)[NW], u32 bits) { nresh += bits; pass64<NW>(s, r, nx); }
    __device__ __forceinline__ u64 reshare1(u64 v, u32 bits) { u64 s[1] = { v }, r[1]; nresh += bits; pass64<1>(s, r, nx); return r[0]; }
    __device__ __forceinline__ u64 open1(u64 v, u32 bits) { u64 s[1] = { v }, r[1]; nopen += bits; pass64<1>(s, r, pv); return r[0]; }
    template <int NW> __device__ __forceinline__ void open64(const u64 (&s)[NW], u64 (&r)[NW]) { pass64<NW>(s, r, pv); }
    __device__ __forceinline__ void drain()
    {
        if (real && nopen) atomicAdd((unsigned long long *)&cnt[2 * p], (unsigned long long)nopen);
        if (real && nresh) atomicAdd((unsigned long long *)&cnt[2 * p + 1], (unsigned long long)nresh);
        nopen = 0; nresh = 0;
    }
    // end of the wavefront: its sums to the context's counters (see LWire::flush)
    __device__ __forceinline__ void flush(u64 *g)
    {
        drain();
        wave_sync();
        const u32 l = threadIdx.x & (GT_LANES - 1);
        if (l < 6) {
            const u64 v = cnt[l];
            if (v) atomicAdd((unsigned long long *)&g[6 * (blockIdx.x & (GT_WIRE_SLOTS - 1)) + l], (unsigned long long)v);
        }
    }
};

// The wavefront model for the per-element protocols where their chain counts and not the vector unit: a row of 16 lanes is 5
// elements x 3 parties (lane 16 r + 5 p + j: party p of element 5 r + j; the row's last lane repeats its first and
// neither stores nor counts), so that a message is a copy from lane to lane inside a row, two DPP moves a dword and no LDS
// latency: about 30 cycles instead of 150.  Training of 267 x 22, depth 4, 473 -> 463 us; of 1,200 x 60, depth 6, 738 -> 720 us.
// Chosen by kernel, not by launch: PRF_ALONE, without issue priorities, where the launches are small as a rule (the arg-max, the
// updates, one-hots, labels, completions of sums, Boolean tests, divisions and scores with four wavefronts per tile), whatever their size.  On a
// full chip the lane moves still cost no more than LDS does: 10,001 wavefronts of k_dot_fin 14.2 us (through LDS 14.4), 14,746 of k_count_fin
// 22.7 (22.7), 7,374 of k_update 17.5 (19.4), 4,096 of k_argmax<1> 18.3 (18.4); through LDS with priorities 13.0, 20.0, 18.1 and 15.4, and
// 2 to 8 % more than DPP where SIMDs have one wavefront.
struct DWire : WWire {
    __device__ __forceinline__ void init(uint4 *region, u64 *s_cnt)
    {
        const u32 l = threadIdx.x & (GT_LANES - 1), x = l & 15;
        real = x < 15; m = l;
        p = x == 15 ? 0 : (int)(x / 5); pn = p == 2 ? 0 : p + 1;
        t = (l >> 4) * 5 + (x == 15 ? 0 : x - 5 * (u32)p);
        nx = 0; pv = 0;
        buf = region; cnt = s_cnt; nopen = 0; nresh = 0;
        if (l < 6) cnt[l] = 0;
        wave_sync();
    }
    __device__ __forceinline__ u32 lane_of(u32 e) const { return e / 5 * 16 + 5 * (u32)p + e % 5; }
    // from the next party's lane, 5 on in the row's 15; from the previous one's, 10 on
    static __device__ __forceinline__ u32 from_next(u32 v)
    {
        const u32 w = (u32)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x110 + 10, 0xf, 0xf, false);          // lanes 10-14: lane - 10
        return (u32)__builtin_amdgcn_update_dpp((int)w, (int)v, 0x100 + 5, 0xf, 0xf, false);                  // lanes 0-10: lane + 5 (15 is as 0)
    }
    static __device__ __forceinline__ u32 from_prev(u32 v)
    {
        const u32 w = (u32)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x100 + 10, 0xf, 0xf, false);          // lanes 0-5: lane + 10 (15 is as 0)
        return (u32)__builtin_amdgcn_update_dpp((int)w, (int)v, 0x110 + 5, 0xf, 0xf, false);                  // lanes 5-15: lane - 5
    }
    static __device__ __forceinline__ u64 join(u32 lo, u32 hi) { return (u64)lo | ((u64)hi << 32); }
    template <int NW>
    __device__ __forceinline__ void reshare(const u64 (&s)[NW], u64 (&r)[NW], u32 bits)
    {
        nresh += bits;
#pragma unroll
        for (int j = 0; j < NW; j++) r[j] = join(from_next((u32)s[j]), from_next((u32)(s[j] >> 32)));
    }
    __device__ __forceinline__ u64 reshare1(u64 v, u32 bits) { u64 s[1] = { v }, r[1]; reshare<1>(s, r, bits); return r[0]; }
    __device__ __forceinline__ u64 open1(u64 v, u32 bits) { nopen += bits; return join(from_prev((u32)v), from_prev((u32)(v >> 32))); }
};
template <int ISSUE> struct ElWire { typedef WWire T; };
template <> struct ElWire<PRF_ALONE> { typedef DWire T; };

// keys of the wavefront model: the lane's own pairwise key in vector registers (the words
// under its next key come from the next party's lane), the dealer's key in scalar ones
__device__ __forceinline__ Key load_lane_key(const u32 *keys, int p)
{
    Key k;
#pragma unroll
    for (int i = 0; i < 8; i++) k.k[i] = keys[p * 8 + i];
    return k;
}

// ---------------------------------------------------------------------------------
// Per-element protocols in the wavefront model: a tile of at most 20 consecutive elements, one
// per lane of a party.  One pass of the block function yields everything a step of the tile
// needs: the dealer blocks of the elements (their components go to all three parties) and, for
// NS streams, the words under the three pairwise keys of the three groups of 8 elements that
// the tile can touch ((e0 mod 8) + elements <= 24); 20 + 9*NS <= 63 lanes.  With a party per
// wavefront every party evaluated the same dealer blocks and a pass per one or two streams
// kept 16 or 32 of 64 lanes busy: three passes for 21 elements instead of one.
#define GT_EL 20
#define GT_EL_WORDS(NS) (10 * GT_TP + (NS) * 3 * 24 + 4)      // (+ 4: idle lanes load up to four words past the last stream's)
template <int NS, int ISSUE = PRF_ALONE>
struct ElTile {
    static_assert(GT_EL + 9 * NS <= 3 * GT_TP, "more blocks than lanes");
    // The lane's block is the dealer's (m < GT_EL: element m) or, with m - GT_EL = 9 i + 3 j + g, stream i, key j, group g.  Its key stays in
    // registers in the kernels without issue priorities (267 x 22, depth 4: 436 us, 430 so; 267 tiles of scores 24.3 and 23.2; on a full chip, too:
    // 2,456 tiles of k_dot_fin 8.4 and 8.2, 15,104 of k_count_fin 27.0 and 26.3, 7,553 of k_update 22.8 and 22.3, 4,096 nodes of k_argmax<1> 47 and 41);
    // in the others the registers are worth more (100,003 quotients 75 us, 83 so) and it is fetched for every block.
    static constexpr bool HELD = ISSUE == PRF_ALONE;
    Key held;
    const u32 *keys;
    u32 role;                    // m - GT_EL
    u64 *mat;                    // GT_EL_WORDS(NS) words: [10][21] dealer components, [NS][3][24] words
    __device__ __forceinline__ Key fetch(int key) const
    {
        Key k;
#pragma unroll
        for (int q = 0; q < 8; q++) k.k[q] = keys[key * 8 + q];
        return k;
    }
    __device__ __forceinline__ void init(const u32 *keys_, const WWire &W, u64 *mat_)
    {
        keys = keys_; mat = mat_;
        role = W.m - GT_EL;
        if (HELD) held = fetch(W.m < GT_EL ? GT_KEY_DEALER : (int)((role % 9) / 3));
    }
    // nel_d: elements of the tile that need the dealer's words (0: none)
    __device__ __forceinline__ void deal(const WWire &W, u32 op, u64 e0, const u32 (&st)[NS], u32 nel_d)
    {
        const u32 m = W.m, r = HELD ? role : m - GT_EL, i = r / 9, j = (r % 9) / 3, g = r % 3;
        const bool dealer = m < GT_EL;
        wave_sync();
        if (dealer ? m < nel_d : r < 9 * NS) {
            const Key kv = HELD ? held : fetch(dealer ? GT_KEY_DEALER : (int)j);
            u32 stream = 0;
#pragma unroll
            for (int q = 0; q < NS; q++) stream = !dealer && i == (u32)q ? st[q] : stream;
            u64 D[8];
            chacha8<ISSUE>(kv, dealer ? e0 + m : (e0 >> 3) + g, op, stream, D);
            if (dealer) {
                const u64 beta = D[5] & 1;
                const u32 b0 = (u32)(D[5] >> 1) & 1, b1 = (u32)(D[5] >> 2) & 1;
                mat[m] = D[1]; mat[GT_TP + m] = D[2]; mat[2 * GT_TP + m] = D[0] - D[1] - D[2];
                mat[3 * GT_TP + m] = D[3]; mat[4 * GT_TP + m] = D[4]; mat[5 * GT_TP + m] = D[0] ^ D[3] ^ D[4];
                mat[6 * GT_TP + m] = D[6]; mat[7 * GT_TP + m] = D[7]; mat[8 * GT_TP + m] = beta - D[6] - D[7];
                mat[9 * GT_TP + m] = b0 | (b1 << 1) | ((((u32)beta ^ b0 ^ b1) & 1) << 2);
            } else {
#pragma unroll
                for (int q = 0; q < 8; q++) mat[10 * GT_TP + (HELD ? r * 8 : (i * 3 + j) * 24 + g * 8) + q] = D[q];
            }
        }
        wave_sync();
    }
    // a single stream, the first (the words of further ones, where the tile has room for them, are not used)
    __device__ __forceinline__ void deal_mask(const WWire &W, u32 op, u64 e0, u32 stream, u32 nel_d)
    {
        u32 st[NS];
#pragma unroll
        for (int q = 0; q < NS; q++) st[q] = stream;
        deal(W, op, e0, st, nel_d);
    }
    // party W.p's components of the tile's element W.t
    __device__ __forceinline__ Dealer dealer(const WWire &W) const
    {
        Dealer D;
        const u64 *m = mat + W.t;
        const u32 b = (u32)m[9 * GT_TP];
        D.rA.o = m[W.p * GT_TP]; D.rA.n = m[W.pn * GT_TP];
        D.rho.o = m[(3 + W.p) * GT_TP]; D.rho.n = m[(3 + W.pn) * GT_TP];
        D.bA.o = m[(6 + W.p) * GT_TP]; D.bA.n = m[(6 + W.pn) * GT_TP];
        D.bBo = (b >> W.p) & 1; D.bBn = (b >> W.pn) & 1;
        return D;
    }
    // words of the i-th stream under the party's two keys; w: (e0 mod 8) + number of the element in the tile
    __device__ __forceinline__ u64 za(const WWire &W, int i, u32 w) const
    { const u64 *m = mat + 10 * GT_TP + i * 72 + w; return m[W.p * 24] - m[W.pn * 24]; }
    __device__ __forceinline__ u64 zb(const WWire &W, int i, u32 w) const
    { const u64 *m = mat + 10 * GT_TP + i * 72 + w; return m[W.p * 24] ^ m[W.pn * 24]; }
};

// Tiles of NEL elements (a multiple of 8), two per lane of a party, for launches that fill the chip: a tile starts at a multiple of 8, so that its
// words under the three keys are whole blocks, 3 NEL / 8 a stream, and NEL dealer blocks and these make up one pass of the block function
// (40 elements and one stream: 55 of 63 lanes, where ElTile's 20 leave 34 idle).
template <int NEL, int NS>
struct ElPair {
    static constexpr int G = NEL / 8, L = NEL / 2;      // blocks of a stream and key, lanes of a party
    static constexpr int ROW = NEL + (L + 32 - NEL % 32) % 32;           // words of a row: L modulo 32, the parties' loads in other banks
    static_assert(NEL + 3 * G * NS <= 3 * GT_TP && L <= GT_TP && ROW % 32 == L, "more blocks than lanes");
    static constexpr int WORDS = (10 + 3 * NS) * ROW;   // [10] dealer components, [NS][3] words
    const u32 *keys;
    u64 *mat;
    __device__ __forceinline__ void deal(const WWire &W, u32 op, u64 e0, const u32 (&st)[NS], u32 nel)
    {
        const u32 m = W.m, r = m - NEL, q = r / G, g = r % G;           // q = 3 i + j: stream i, key j
        const bool dealer = m < NEL;
        wave_sync();
        if (dealer ? m < nel : r < 3 * G * NS) {
            Key k;
            const u32 *from = keys + 8 * (dealer ? GT_KEY_DEALER : q % 3);
#pragma unroll
            for (int i = 0; i < 8; i++) k.k[i] = from[i];
            u32 stream = 0;
#pragma unroll
            for (int i = 0; i < NS; i++) stream = !dealer && q / 3 == (u32)i ? st[i] : stream;
            u64 D[8];
            chacha8<PRF_PAIR>(k, dealer ? e0 + m : (e0 >> 3) + g, op, stream, D);
            if (dealer) {
                const u64 beta = D[5] & 1;
                const u32 b0 = (u32)(D[5] >> 1) & 1, b1 = (u32)(D[5] >> 2) & 1;
                mat[m] = D[1]; mat[ROW + m] = D[2]; mat[2 * ROW + m] = D[0] - D[1] - D[2];
                mat[3 * ROW + m] = D[3]; mat[4 * ROW + m] = D[4]; mat[5 * ROW + m] = D[0] ^ D[3] ^ D[4];
                mat[6 * ROW + m] = D[6]; mat[7 * ROW + m] = D[7]; mat[8 * ROW + m] = beta - D[6] - D[7];
                mat[9 * ROW + m] = b0 | (b1 << 1) | ((((u32)beta ^ b0 ^ b1) & 1) << 2);
            } else {
#pragma unroll
                for (int i = 0; i < 8; i++) mat[(10 + q) * ROW + 8 * g + i] = D[i];
            }
        }
        wave_sync();
    }
    __device__ __forceinline__ Dealer dealer(const WWire &W, u32 e) const
    {
        Dealer D;
        const u64 *m = mat + e;
        const u32 b = (u32)m[9 * ROW];
        D.rA.o = m[W.p * ROW]; D.rA.n = m[W.pn * ROW];
        D.rho.o = m[(3 + W.p) * ROW]; D.rho.n = m[(3 + W.pn) * ROW];
        D.bA.o = m[(6 + W.p) * ROW]; D.bA.n = m[(6 + W.pn) * ROW];
        D.bBo = (b >> W.p) & 1; D.bBn = (b >> W.pn) & 1;
        return D;
    }
    // the Boolean zero-sharing word of stream i
    __device__ __forceinline__ u64 zb(const WWire &W, int i, u32 e) const { return mat[(10 + 3 * i + W.p) * ROW + e] ^ mat[(10 + 3 * i + W.pn) * ROW + e]; }
};

// [v == 0] of a lane's two elements: the rounds of eq_bit_mask, a dword for both from the second on; the result's bits 0 and 16.
// na: how many of the two exist.
__device__ __forceinline__ void eq_bits2(WWire &W, const Sh (&v)[2], const Dealer (&D)[2], const u64 (&A)[2], u32 na, u32 &ro, u32 &rn)
{
    const u32 M0 = W.p == 0 ? ~0u : 0u, M2 = W.p == 2 ? ~0u : 0u;
    u64 snd[2], rcv[2];
    u32 x[2], y[2], H[2];
#pragma unroll
    for (int h = 0; h < 2; h++) snd[h] = v[h].o + D[h].rA.o;
    W.open64<2>(snd, rcv);
#pragma unroll
    for (int h = 0; h < 2; h++) {
        const u64 c = snd[h] + v[h].n + D[h].rA.n + rcv[h];
        const u32 cl = (u32)c, ch = (u32)(c >> 32);
        // t = rho with the complement of c xored into component 0
        const u32 tol = logic3<0xd2>((u32)D[h].rho.o, cl, M0), toh = logic3<0xd2>((u32)(D[h].rho.o >> 32), ch, M0);
        const u32 tnl = logic3<0xd2>((u32)D[h].rho.n, cl, M2), tnh = logic3<0xd2>((u32)(D[h].rho.n >> 32), ch, M2);
        x[h] = and3l(tol, tnl, toh, tnh) ^ (u32)A[h];
        H[h] = (u32)(A[h] >> 32);
    }
    W.reshare<2>(x, y);
    const u32 LO = 0x05040100u, HI = 0x07060302u;               // halves of a pair of dwords
    u32 P[1] = { and3l(__builtin_amdgcn_perm(x[1], x[0], LO), __builtin_amdgcn_perm(y[1], y[0], LO), __builtin_amdgcn_perm(x[1], x[0], HI), __builtin_amdgcn_perm(y[1], y[0], HI))
                 ^ __builtin_amdgcn_perm(H[1], H[0], LO) }, Q[1];
    u32 B = __builtin_amdgcn_perm(H[1], H[0], HI);              // bits 48-63 of the mask words
    W.reshare<1>(P, Q);
#pragma unroll
    for (int i = 0; i < 4; i++) {
        const int w = 8 >> i;
        P[0] = logic3<0x60>(w == 8 ? 0x00ff00ffu : w == 4 ? 0x000f000fu : w == 2 ? 0x00030003u : 0x00010001u, and3l(P[0], Q[0], P[0] >> w, Q[0] >> w), B);
        W.reshare<1>(P, Q);
        B >>= w;
    }
    W.nopen += 64u * na; W.nresh += 63u * na;
    ro = P[0]; rn = Q[0];
}
