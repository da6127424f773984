// pairs.h -- the endgame DAG of two roots at once (Section VIII), for roots
// with up to 8 empty cells.
//
// Two roots with the same number of empty cells have the same DAG: the same
// nodes, children and five-set subsets.  They are solved together, their sets
// side by side in the same words, so that the node and child indices are
// worked out once, and in a layout where rmax needs no shifts and masks.
//
// Write g_j = p_j + 2 h_j.  The neighbours g_j +- 1 of g_j are the two values
// of h_j at the other p_j, so along one dimension rmin is "AND the two h_j,
// and exchange the two p_j".  Two quantities never mix.  The chain: a node's
// win set comes from its children's not-lose sets and the other way round, so
// following win at even and not-lose at odd layers (chain 0) or the reverse
// (chain 1) gives two independent solves.  And the parity s of
// p_0 + p_1 + p_2 + p_3 + t over the layers t, since a turn changes one p_j
// and a placement leads to the next layer.  So a position's 512 bits for
// layer t are kept as
//   lane of a quad: h2 + 2 h3
//   register k:     p1 + 2 p2 + 4 p3
//   bit:            s + 2 chain + 4 root + 8 h1 + 16 h0   (p0 follows from s)
// and rmin is, per register, two ANDs with a quad neighbour (h2, h3), two
// with the word's own bytes exchanged (h1, h0), taken from the registers
// with one p_j flipped (dimension 0 flips p0, which is implied by s at the
// next layer): 7 instructions for 32 bits, against 17 in the layout of
// Set256, where the p_j of dimensions 0 and 1 are bits of the same word.
//
// What bounds it: VALU issue and LDS reads alike (8 empty cells, one 1024-thread
// workgroup per CU: 0.60 of the issue peak; an LDS instruction in 19 cycles, of
// the 8 that 16 bytes a lane take, and bank conflicts in 0.15 of the cycles);
// the layers' barriers leave the rest.  ns per root, 131,072 roots of one
// size, against one root per workgroup or wave in the layout of Set256:
//   empty cells    3      4      5      6      7      8
//   one root      2.42   3.92   6.99  13.84  28.79  77.76
//   pairs         1.12   1.84   3.32   6.33  12.54  33.05
//
// A node's record for its parents is the complement of its prepared terms,
// ~F_o & rmin(X) for X = win or not-lose: parents AND their children's.
#pragma once
#include "device_common.h"

namespace pg {

constexpr int binom_c(int n, int k)
{
    if (k < 0 || k > n) return 0;
    int r = 1;
    for (int i = 1; i <= k; i++) r = r * (n - k + i) / i;
    return r;
}

// Sizes of the DAG of E empty cells: t stones placed, ceil(t/2) by the side
// to move at the root (the mover) and floor(t/2) by the other side.
template <int E>
struct PairDag {
    static constexpr int nodes(int t) { return binom_c(E, t) * binom_c(t, t / 2); }
    static constexpr int layer_start(int t)
    {
        int n = 0;
        for (int i = 0; i < t; i++) n += nodes(i);
        return n;
    }
    static constexpr int max_layer()
    {
        int n = 0;
        for (int t = 0; t <= E; t++) n = nodes(t) > n ? nodes(t) : n;
        return n;
    }
    // subsets of the cells with fewer than s elements
    static constexpr int below(int s)
    {
        int n = 0;
        for (int i = 0; i < s; i++) n += binom_c(E, i);
        return n;
    }
    static constexpr int fives_c = below((E + 1) / 2 + 1);          // five-sets of the mover: sizes 0..ceil(E/2)
    static constexpr int fives = fives_c + below(E / 2 + 1);        // then the other side's: 0..floor(E/2)
    // LDS of one pair, in uint4: the records of one layer (also the first
    // form of the five-sets, 4 uint4 per subset), the five-sets, the roots
    static constexpr int rec_u4 = 8 * max_layer() > 4 * fives ? 8 * max_layer() : 4 * fives;
    static constexpr int five_u4 = 16 * fives;
    static constexpr int root_u4 = 12;
    static constexpr int lds_bytes = 16 * (rec_u4 + five_u4 + root_u4);
};

// The two roots of a pair in LDS: per root the stones of the mover and of the
// other side as two 18-bit masks (quadrants 0 and 1, quadrants 2 and 3), and
// the mask of each empty cell.
struct PairRoot {
    uint2 own, other;
    uint2 slot[10];
};
static_assert(2 * sizeof(PairRoot) == 16 * PairDag<8>::root_u4, "PairRoot");

// bitwise operations of three words in one instruction
__device__ __forceinline__ uint32_t and3(uint32_t a, uint32_t b, uint32_t c)
{
    return (uint32_t)__builtin_amdgcn_bitop3_b32(a, b, c, 0x80);
}
__device__ __forceinline__ uint32_t andn3(uint32_t n, uint32_t b, uint32_t c)  // ~n & b & c
{
    return (uint32_t)__builtin_amdgcn_bitop3_b32(n, b, c, 0x08);
}

// exchange adjacent bits
__device__ __forceinline__ uint32_t swap_bit0(uint32_t x) { return bfi(0x55555555u, x >> 1, x << 1); }

__device__ __forceinline__ void unpack8(uint32_t (&w)[8], const uint4 a, const uint4 b)
{
    w[0] = a.x; w[1] = a.y; w[2] = a.z; w[3] = a.w;
    w[4] = b.x; w[5] = b.y; w[6] = b.z; w[7] = b.w;
}

// x AND x of the quad lane whose number differs by X (1 or 2)
template <int X>
__device__ __forceinline__ uint32_t and_quad(uint32_t x)
{
    return x & quad_perm<X == 1 ? 0xB1 : 0x4E>(x);
}

// ~fo & rmin(u) (see above)
__device__ __forceinline__ void pair_record(uint32_t (&r)[8], const uint32_t (&u)[8], const uint32_t (&fo)[8])
{
    uint32_t y2[8], y3[8];
#pragma unroll
    for (int k = 0; k < 8; k++) {
        y2[k] = and_quad<1>(u[k]);
        y3[k] = and_quad<2>(u[k]);
    }
#pragma unroll
    for (int k = 0; k < 8; k++) {
        const uint32_t a = u[k], b = u[k ^ 1];
        const uint32_t ah = rotr32(a, 16);                                                // h0 exchanged
        const uint32_t bh = (uint32_t)__builtin_amdgcn_perm(b, b, 0x02030001u);           // h1 exchanged
        r[k] = andn3(fo[k], and3(a, ah, y2[k ^ 2]), and3(b, bh, y3[k ^ 4]));
    }
}

// The edge records of a lane's nodes of layer t (their first halves hold the
// children of up to 6 free cells), loaded a layer ahead: behind the barrier
// their latency would stand in every layer's chain.
template <int E, int T_, int GL>
struct PairEdges {
    static constexpr int passes = (4 * PairDag<E>::nodes(T_) + GL - 1) / GL;
    uint4 a[passes], b[passes];
    __device__ __forceinline__ void load(const uint4 *edges, int gl)
    {
        constexpr int n = PairDag<E>::nodes(T_);
#pragma unroll
        for (int p = 0; p < passes; p++) {
            const int it = gl + p * GL;
            if ((p + 1) * GL <= 4 * n || it < 4 * n) {
                const uint4 *ed = edges + 2 * (PairDag<E>::layer_start(T_) + (it >> 2));
                a[p] = ed[0];
                if (E - T_ > 6) b[p] = ed[1];
            }
        }
    }
};

// One layer of a pair's DAG: `gl` is the lane's number among the GL threads
// of the pair (quads of lanes share a node).  rec: records [2][max_layer][4
// lanes] of 4 registers each; five: [2 parities of t][2][fives][4].  Every
// lane holds its results until all children are read: one layer buffer.
template <int E, int T_, int GL>
__device__ __forceinline__ void pair_layer(const uint4 *edges, uint4 *rec, const uint4 *five, int gl,
                                           const PairEdges<E, T_, GL> &mine)
{
    using D = PairDag<E>;
    constexpr int t = T_, n = D::nodes(t), passes = PairEdges<E, T_, GL>::passes, nfree = E - t;
    constexpr uint32_t winner = (t & 1) ? 0xccccccccu : 0x33333333u;  // the chain that holds win sets here
    constexpr int ML = D::max_layer(), NF = D::fives;
    const int q = gl & 3;
    uint32_t r[passes][8];
#pragma unroll
    for (int p = 0; p < passes; p++) {
        const int it = gl + p * GL;
        if ((p + 1) * GL <= 4 * n || it < 4 * n) {
            const uint4 ea = mine.a[p];
            uint4 eb = make_uint4(0, 0, 0, 0);
            if (nfree > 6) eb = mine.b[p];
            const uint32_t w[8] = {ea.x, ea.y, ea.z, ea.w, eb.x, eb.y, eb.z, eb.w};
            const int ic = 4 * (D::below((t + 1) / 2) + (int)(w[0] & 0xffffu)) + q;
            const int io = 4 * (D::fives_c + D::below(t / 2) + (int)(w[0] >> 16)) + q;
            const int ix = (t & 1) ? io : ic, iy = (t & 1) ? ic : io;
            const uint4 *fx = five + (t & 1) * 8 * NF + ix, *fy = five + (t & 1) * 8 * NF + iy;
            uint32_t X[8], Fx[8], Fy[8], a[8];
            unpack8(Fx, fx[0], fx[4 * NF]);
            unpack8(Fy, fy[0], fy[4 * NF]);
            if (nfree == 0) {
#pragma unroll
                for (int k = 0; k < 8; k++) a[k] = winner;
            } else {
#pragma unroll
                for (int c = 0; c < nfree; c += 2) {
                    const uint32_t c0 = (w[1 + (c >> 1)]) & 0xffffu, c1 = w[1 + (c >> 1)] >> 16;
                    uint32_t u[8], v[8];
                    const uint4 *pu = rec + 4 * c0 + q;
                    unpack8(u, pu[0], pu[4 * ML]);
                    if (c + 1 < nfree) {
                        const uint4 *pv = rec + 4 * c1 + q;
                        unpack8(v, pv[0], pv[4 * ML]);
                    }
#pragma unroll
                    for (int k = 0; k < 8; k++) {
                        if (c + 1 < nfree) a[k] = c == 0 ? u[k] & v[k] : and3(a[k], u[k], v[k]);
                        else a[k] = c == 0 ? u[k] : a[k] & u[k];
                    }
                }
            }
#pragma unroll
            for (int k = 0; k < 8; k++) {
                // win: ~Fy & (Fx | ~a), not-lose: Fx | (~Fy & ~a)
                const uint32_t g = (uint32_t)__builtin_amdgcn_bitop3_b32(Fx[k], Fy[k], winner, 0x70);  // Fx & ~(Fy & winner)
                X[k] = (uint32_t)__builtin_amdgcn_bitop3_b32(g, Fy[k], a[k], 0xf1);                    // g | ~(Fy | a)
            }
            if constexpr (t == 0) {
#pragma unroll
                for (int k = 0; k < 8; k++) r[p][k] = X[k];
            } else {
                // the record belongs to the next layer: its five-set in that parity's form
                const uint4 *fz = five + ((t - 1) & 1) * 8 * NF + iy;
                uint32_t Fz[8];
                unpack8(Fz, fz[0], fz[4 * NF]);
                pair_record(r[p], X, Fz);
            }
        }
        // one pass after another: interleaved, their registers spill
        __builtin_amdgcn_sched_barrier(0);
    }
    PairEdges<E, t == 0 ? 0 : t - 1, GL> next;
    if constexpr (t > 0) {
        next.load(edges, gl);
        __syncthreads();
    }
#pragma unroll
    for (int p = 0; p < passes; p++) {
        const int it = gl + p * GL;
        if ((p + 1) * GL <= 4 * n || it < 4 * n) {
            rec[it] = make_uint4(r[p][0], r[p][1], r[p][2], r[p][3]);
            rec[4 * ML + it] = make_uint4(r[p][4], r[p][5], r[p][6], r[p][7]);
        }
    }
    __syncthreads();
    if constexpr (t > 0) pair_layer<E, t - 1, GL>(edges, rec, five, gl, next);
}

// Solve PAIRS pairs of roots with E empty cells by a workgroup of NT threads
// (NT / PAIRS, at least 32, each): board[0], board[1] and out[0], out[1] are
// this thread's pair's (a pair may name one root twice).  Every thread of the
// workgroup calls it; lds holds PAIRS * PairDag<E>::lds_bytes.
template <int E, int NT, int PAIRS>
__device__ void solve_pairs(const uint64_t (&board)[2], uint4 *const (&out)[2], const DevTables &T, uint4 *lds)
{
    using D = PairDag<E>;
    constexpr int GL = NT / PAIRS, ML = D::max_layer(), NF = D::fives;
    static_assert(GL >= 32 && GL % 32 == 0, "a pair's output takes 32 lanes");
    int gl = (int)threadIdx.x % GL;
    // opaque: the addresses of every layer's passes depend on gl alone, and
    // kept in registers from root to root they spill
    asm volatile("" : "+v"(gl));
    uint4 *rec = lds + (threadIdx.x / GL) * (D::lds_bytes / 16);
    uint4 *five = rec + D::rec_u4;
    PairRoot *root = (PairRoot *)(five + D::five_u4);
    if (gl < 8) {
        // lane 4 r + j: quadrant j of root r (E even: black moves)
        const int r = gl >> 2, j = gl & 3;
        int x = (int)((board[r] >> (16 * j)) & 0xffffu);
        unsigned bm = 0, wm = 0;
#pragma unroll
        for (int l = 0; l < 9; l++) {
            const int d = x % 3;
            x /= 3;
            bm |= (unsigned)(d == 1) << l;
            wm |= (unsigned)(d == 2) << l;
        }
        unsigned em = ~(bm | wm) & 0x1ffu;
        const int cnt = __popc(em);
        // empty cells of the quadrants before this one
        int first = 0;
#pragma unroll
        for (int i = 0; i < 3; i++) {
            const int c = __shfl(cnt, (int)(threadIdx.x & 60u) + i, 64);
            first += i < j ? c : 0;
        }
        const int sh = 9 * (j & 1);
        uint32_t *own = (uint32_t *)&root[r].own + (j >> 1), *other = (uint32_t *)&root[r].other + (j >> 1);
        const unsigned mine = (E & 1) ? wm : bm, theirs = (E & 1) ? bm : wm;
        // the two quadrants of a mask are joined by the even one's lane
        const unsigned mine_hi = quad_perm<0xB1>(mine), theirs_hi = quad_perm<0xB1>(theirs);
        if ((j & 1) == 0) {
            *own = mine | (mine_hi << 9);
            *other = theirs | (theirs_hi << 9);
        }
        for (int k = first; em; k++) {
            const unsigned bit = em & (0u - em);
            em ^= bit;
            root[r].slot[k] = j < 2 ? make_uint2(bit << sh, 0u) : make_uint2(0u, bit << sh);
        }
    }
    __syncthreads();
    // five-sets, one subset of one root per lane, in the words of SplitBits
    const uint16_t *smask = T.dag_sub_mask + T.dag_sub_off[E];
    for (int it = gl; it < 2 * NF; it += GL) {
        const int r = it >= NF, i = it - (r ? NF : 0);
        const bool mine = i < D::fives_c;
        const uint32_t m = smask[mine ? i : i - D::fives_c];
        const uint2 base = mine ? root[r].own : root[r].other;
        uint32_t lo = base.x, hi = base.y;
#pragma unroll
        for (int sl = 0; sl < E; sl++) {
            const uint2 c = root[r].slot[sl];
            const uint32_t on = (uint32_t)((int)(m << (31 - sl)) >> 31);
            lo |= c.x & on;
            hi |= c.y & on;
        }
        const Set256 F = five_set<SplitBits>(T.lm[lo & 511u], T.lm[512 + (lo >> 9)], T.lm[1024 + (hi & 511u)],
                                             T.lm[1536 + (hi >> 9)]);
        uint4 *dst = rec + 4 * i + 2 * r;
        dst[0] = make_uint4(F.w[0], F.w[1], F.w[2], F.w[3]);
        dst[1] = make_uint4(F.w[4], F.w[5], F.w[6], F.w[7]);
    }
    __syncthreads();
    // both roots' five-sets into the registers and bits of the layer solve,
    // once for even and once for odd layers (s and p0 exchange meaning)
    for (int it = gl; it < 4 * NF; it += GL) {
        const int q = it & 3;
        const uint32_t *src = (const uint32_t *)(rec + 4 * (it >> 2)) + (q & 1) + 4 * (q >> 1);
        uint32_t even[8], odd[8];
#pragma unroll
        for (int p3 = 0; p3 < 2; p3++) {
            const uint32_t w0 = src[2 * p3], w1 = src[8 + 2 * p3];
#pragma unroll
            for (int p2 = 0; p2 < 2; p2++) {
                // p0, p1 of root 0 at bits 0, 1 and of root 1 at bits 2, 3 of a byte's halves
                const uint32_t u = p2 ? bfi(0x0f0f0f0fu, w0 >> 4, w1) : bfi(0x0f0f0f0fu, w0, w1 << 4);
#pragma unroll
                for (int p1 = 0; p1 < 2; p1++) {
                    const uint32_t z = p1 ? bfi(0x33333333u, u >> 2, u) : bfi(0xccccccccu, u << 2, u);
                    const uint32_t y = swap_bit0(z);
                    const int k = p1 + 2 * p2 + 4 * p3;
                    const bool flip = ((p1 + p2 + p3) & 1) != 0;
                    even[k] = flip ? y : z;
                    odd[k] = flip ? z : y;
                }
            }
        }
        uint4 *dst = five + it;
        dst[0] = make_uint4(even[0], even[1], even[2], even[3]);
        dst[4 * NF] = make_uint4(even[4], even[5], even[6], even[7]);
        dst[8 * NF] = make_uint4(odd[0], odd[1], odd[2], odd[3]);
        dst[12 * NF] = make_uint4(odd[4], odd[5], odd[6], odd[7]);
    }
    const uint4 *edges = T.dag_edge + 2 * T.dag_node_off[E];
    PairEdges<E, E, GL> first;
    first.load(edges, gl);
    __syncthreads();
    pair_layer<E, E, GL>(edges, rec, five, gl, first);
    // the root's win and not-lose sets back into the words of Set256: lane
    // w + 8 chain + 16 root takes word w = h2 + 2 p3 + 4 h3
    if (gl < 32) {
        const int w = gl & 7, h2 = w & 1, p3 = (w >> 1) & 1, h3 = w >> 2, sh = 2 * ((gl >> 3) & 1) + 4 * (gl >> 4);
        const uint4 x = rec[4 * ML * p3 + h2 + 2 * h3];
        const uint32_t v[4] = {x.x, x.y, x.z, x.w};
        uint32_t o = 0;
#pragma unroll
        for (int k = 0; k < 4; k++) {
            uint32_t b = (v[k] >> sh) & 0x03030303u;
            const uint32_t y = swap_bit0(b);
            b = (((k ^ (k >> 1)) ^ p3) & 1) ? y : b;
            o |= ((b & 0x0303u) | ((b >> 14) & 0x0c0cu)) << (4 * (k & 1) + 16 * (k >> 1));
        }
        uint32_t *dst = (uint32_t *)(gl < 16 ? out[0] : out[1]);
        dst[gl & 15] = o;
    }
    __syncthreads();
}

}  // namespace pg
