// deep.hip -- the endgame solver for one deep root (Section VIII: positions
// outside the database are solved from scratch, rotations folded in by rmax
// only; the paper's serial solver evaluates an 18-stone position in 16 s on
// one CPU thread).  Where the batched solver keeps a root's whole DAG in one
// workgroup's LDS (up to 10 empty cells), this one spreads each layer of one
// root over the whole GPU, with the layers in HBM: an 18-empty root has
// 86,574,831 nodes, at most 17,153,136 in one layer.
//
// Node (t, cmask, omask) of a root with e empty cells is the root with t more
// stones: the root's side to move (the mover) on the cells of cmask (ceil(t/2)
// of them), the other side on omask (floor(t/2)), cells numbered 0..e-1.
// Layers are solved from t = e down to 0, each node keeping for its parents a
// record of its prepared terms, two layers at a time.
//
// The whole table (pentago_eval_deep).  At layer t side x places a stone and
// y's stones stay: the children of all nodes with one y mask are the nodes of
// the next layer with that y mask.  So a layer is stored in blocks of one mask
// of the side that does not move at the layer below it (its parents'), and a
// block of parents reads one block of children, each record once from HBM.
// Within a block, which child belongs to which parent depends on the block's
// sizes only: the child numbers come from one table per layer instead of
// from ranking every child (1485 VALU instructions per node, most of them
// ranks, before).  Four lanes share a node and read its records 16 bytes each,
// so an instruction reads 16 whole records.  The record layout is that of
// pairs.h with p3 in the place of the root number: lane h2 + 2 h3, register
// p1 + 2 p2, bit s + 2 chain + 4 p3 + 8 h1 + 16 h0.
//
// One parity (pentago_eval_deep_parity) keeps the plain form: node index in
// layer t rank(cmask) * C(e - |cmask|, |omask|) + rank'(omask), with rank the
// colex rank of a subset of the e cells (sum of C(c_i, i + 1) over its cells
// c_0 < c_1 < ...) and rank' the colex rank of omask among the cells not in
// cmask; a record is A = F_parent(node) | rmax(not N), B = F_parent(node) |
// rmax(not W) at one parity (32 B).
#include "device_common.h"
#include "internal.h"
#include "pairs.h"

#include <algorithm>
#include <cstring>
#include <mutex>
#include <set>

namespace pg {

constexpr int kDeepMaxEmpty = 20;

static __constant__ uint32_t c_binom[kDeepMaxEmpty + 2][kDeepMaxEmpty + 2];

struct DeepJob {
    int e;                        // empty cells of the root
    int t;                        // layer
    int mover;                    // side to move at the root (1 black, 2 white)
    unsigned cm0[4], om0[4];      // the root's stones of the mover and the other side
    int slot_q[kDeepMaxEmpty];    // quadrant and local cell of each empty cell
    int slot_l[kDeepMaxEmpty];
    uint32_t nsub_c, nsub_o;      // subsets of the mover's / other side's size in layer t
    uint32_t nodes;               // nodes of layer t
    uint4 *ftab;                  // five-sets: [nsub_c] of the mover's subsets, then [nsub_o]
    const uint4 *prev;            // A/B records of layer t + 1
    uint4 *cur;                   // A/B records of layer t
    uint4 *out;                   // the root's W/N (t = 0)
    int parity;                   // only the root's g with this parity (0 / 1) of sum g_i
};

// Parity-halved records (Section VIII: rmax flips the parity of
// g0 + g1 + g2 + g3, so a root's values of one parity need each layer's
// terms of one parity only, alternating from layer to layer).  Bit
// g0 + 4 g1 + 16 (g2 & 1) of word (g2 >> 1) + 2 g3 has parity
// popcount(bit & 0x15) + g3 (mod 2); kEvenBits marks the even bits of the
// words with g3 even (0, 1, 4, 5).  Words w and w ^ 2 differ in g3 by one,
// so the bits of one parity of both fit one word: a 256-bit set of that
// parity packs into 4 words, and a node's A/B record into 32 B.
constexpr uint32_t kEvenBits = 0x5a5aa5a5u;

// Mask of the bits of parity par in the words with g3 even.
__device__ __forceinline__ uint32_t parity_bits(int par) { return par ? ~kEvenBits : kEvenBits; }

// Pack the bits of parity par of x (words 0, 1, 4, 5 with 2, 3, 6, 7).
__device__ __forceinline__ uint4 pack_parity(const Set256 &x, int par)
{
    const uint32_t m = parity_bits(par);
    return make_uint4((x.w[0] & m) | (x.w[2] & ~m), (x.w[1] & m) | (x.w[3] & ~m), (x.w[4] & m) | (x.w[6] & ~m),
                      (x.w[5] & m) | (x.w[7] & ~m));
}

// Unpack: both words of a pair take the packed word.  The bits of the other
// parity then hold values of no meaning; every use below is bitwise per g or
// goes through rmax, which reads them only for results of that other parity,
// and those are dropped again when the next record is packed.
__device__ __forceinline__ Set256 unpack_parity(uint4 v)
{
    Set256 x;
    x.w[0] = x.w[2] = v.x;
    x.w[1] = x.w[3] = v.y;
    x.w[4] = x.w[6] = v.z;
    x.w[5] = x.w[7] = v.w;
    return x;
}

typedef uint32_t BinomRow[kDeepMaxEmpty + 2];

__device__ __forceinline__ uint32_t colex_rank(unsigned mask, const BinomRow *bn)
{
    uint32_t r = 0;
    int i = 0;
    while (mask) {
        const int c = __builtin_ctz(mask);
        mask &= mask - 1;
        r += bn[c][i + 1];
        i++;
    }
    return r;
}

// The subset of {0..n-1} with k elements and colex rank r.
__device__ __forceinline__ unsigned colex_unrank(uint32_t r, int k, int n, const BinomRow *bn)
{
    unsigned mask = 0;
    for (int c = n - 1; c >= 0 && k > 0; c--) {
        const uint32_t b = bn[c][k];
        if (r >= b) {
            mask |= 1u << c;
            r -= b;
            k--;
        }
    }
    return mask;
}

// The k-th bit of m placed at the position of the k-th set bit of `within`
// (pdep).
__device__ __forceinline__ unsigned unpack_bits(unsigned m, unsigned within)
{
    unsigned r = 0;
    int i = 0;
    while (within) {
        const int c = __builtin_ctz(within);
        within &= within - 1;
        r |= ((m >> i) & 1u) << c;
        i++;
    }
    return r;
}

// Colex rank of omask among the cells not in cmask (rank of the packed
// subset): omask's cell c sits at c - popcount(cmask below c) among them.
__device__ __forceinline__ uint32_t rank_in_free(unsigned omask, unsigned cmask, const BinomRow *bn)
{
    uint32_t r = 0;
    int i = 0;
    while (omask) {
        const int c = __builtin_ctz(omask);
        omask &= omask - 1;
        r += bn[c - __popc(cmask & ((1u << c) - 1u))][i + 1];
        i++;
    }
    return r;
}

// The binomial table, copied to LDS by each workgroup: the lanes index it
// with different values, and from LDS those reads cost a few cycles instead
// of a dependent memory load each (the ranking loops chain them).
__device__ __forceinline__ const BinomRow *lds_binom(BinomRow *sb)
{
    for (int k = threadIdx.x; k < (kDeepMaxEmpty + 2) * (kDeepMaxEmpty + 2); k += blockDim.x)
        sb[k / (kDeepMaxEmpty + 2)][k % (kDeepMaxEmpty + 2)] = c_binom[k / (kDeepMaxEmpty + 2)][k % (kDeepMaxEmpty + 2)];
    __syncthreads();
    return sb;
}

// Five-set of every subset of the empty cells of the two sizes of layer t
// (the mover's ceil(t/2) cells, the other side's floor(t/2)), indexed by
// colex rank: each node then reads its two.
__global__ void __launch_bounds__(256) deep_five_kernel(DeepJob J, DevTables T)
{
    __shared__ BinomRow sb[kDeepMaxEmpty + 2];
    const BinomRow *bn = lds_binom(sb);
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= J.nsub_c + J.nsub_o) return;
    const bool mine = i < J.nsub_c;
    const int k = mine ? (J.t + 1) >> 1 : J.t >> 1;
    const unsigned m = colex_unrank(mine ? i : i - J.nsub_c, k, J.e, bn);
    unsigned xm[4];
#pragma unroll
    for (int j = 0; j < 4; j++) xm[j] = mine ? J.cm0[j] : J.om0[j];
    for (int sl = 0; sl < J.e; sl++)
        if ((m >> sl) & 1) {
            const int q = J.slot_q[sl];
            const unsigned bit = 1u << J.slot_l[sl];
            xm[0] |= q == 0 ? bit : 0u;
            xm[1] |= q == 1 ? bit : 0u;
            xm[2] |= q == 2 ? bit : 0u;
            xm[3] |= q == 3 ? bit : 0u;
        }
    const Set256 F = board_five(T, xm);
    uint4 *dst = J.ftab + 2 * (size_t)i;
    dst[0] = make_uint4(F.w[0], F.w[1], F.w[2], F.w[3]);
    dst[1] = make_uint4(F.w[4], F.w[5], F.w[6], F.w[7]);
}

// One node of layer t per thread (Section II recurrence on Section III
// tables): OR the children's prepared terms, combine with the node's own
// five-sets, keep the terms its parents read (the root's W/N at t = 0).
// Records of 32 B hold one parity (for the root's parity J.parity).
__global__ void __launch_bounds__(256) deep_half_kernel(DeepJob J, DevTables T)
{
    __shared__ BinomRow sb[kDeepMaxEmpty + 2];
    const BinomRow *bn = lds_binom(sb);
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= J.nodes) return;
    const int e = J.e, t = J.t;
    const int sc = (t + 1) >> 1, so = t >> 1;
    const unsigned all = (1u << e) - 1u;
    const uint32_t per = bn[e - sc][so];
    const uint32_t r1 = i / per, r2 = i - r1 * per;
    const unsigned cmask = colex_unrank(r1, sc, e, bn);
    const unsigned omask = unpack_bits(colex_unrank(r2, so, e - sc, bn), all & ~cmask);
    // (cmask was unranked from r1, so r1 is its colex rank)
    const Set256 Fc = set_from(J.ftab + 2 * (size_t)r1);
    const Set256 Fo = set_from(J.ftab + 2 * ((size_t)J.nsub_c + colex_rank(omask, bn)));
    const bool xroot = (t & 1) == 0;   // the side to move at layer t is the root's mover
    const Set256 &Fx = xroot ? Fc : Fo;
    const Set256 &Fy = xroot ? Fo : Fc;
    Set256 Wnt = s_zero(), Nnt = s_zero();
    if (t == e) {
        Nnt = s_full();
    } else {
        // children: the side to move puts a stone on a free cell
        // child index rank(cmask') * C(e - |cmask'|, |omask'|) + rank of omask'
        // among the cells not in cmask': cmask grows when the root's mover
        // moves, else omask grows and cmask's rank is the same for all children
        const int cso = xroot ? so : so + 1;   // the other side's stones in layer t + 1
        const uint32_t rc = r1;
        const uint32_t per_c = xroot ? bn[e - sc - 1][cso] : bn[e - sc][cso];
        auto child_index = [&](int sl) -> uint32_t {
            const unsigned bit = 1u << sl;
            return xroot ? colex_rank(cmask | bit, bn) * per_c + rank_in_free(omask, cmask | bit, bn)
                         : rc * per_c + rank_in_free(omask | bit, cmask, bn);
        };
        // Every node of the layer has e - t free cells; two children go per
        // step, both loads issued before either is used (an odd count repeats
        // the last child, which OR absorbs).
        const int nch = e - t;
        unsigned f = all & ~(cmask | omask);
        for (int k = 0; k < nch; k += 2) {
            const int sa = __builtin_ctz(f);
            f &= f - 1;
            const uint32_t ca = child_index(sa);
            const int sb = k + 1 < nch ? __builtin_ctz(f) : sa;
            f &= f - 1;
            const uint32_t cb = child_index(sb);
            const uint4 *pa = J.prev + 2 * (size_t)ca, *pb = J.prev + 2 * (size_t)cb;
            const uint4 a0 = pa[0], a1 = pa[1], b0 = pb[0], b1 = pb[1];
            s_or_into(Wnt, unpack_parity(a0));
            s_or_into(Nnt, unpack_parity(a1));
            s_or_into(Wnt, unpack_parity(b0));
            s_or_into(Nnt, unpack_parity(b1));
        }
    }
    Set256 W, N;
    combine(Fx, Fy, Wnt, Nnt, W, N);
    if (t == 0) {
        // the root's entries of the other parity are cleared
        const uint32_t m = parity_bits(J.parity);
#pragma unroll
        for (int w = 0; w < 8; w++) {
            const uint32_t mw = (w & 2) ? ~m : m;
            W.w[w] &= mw;
            N.w[w] &= mw;
        }
        store_info(J.out, W, N);
    } else {
        // a parent at parity p reads this record at p; layer t's records
        // carry the root's parity for odd t and the other one for even t
        Set256 A, B;
        child_terms(Fy, W, N, A, B);
        const int par = J.parity ^ ((t + 1) & 1);
        uint4 *p = J.cur + 2 * (size_t)i;
        p[0] = pack_parity(A, par);
        p[1] = pack_parity(B, par);
    }
}

// ---------------------------------------------------------------------------
// The whole table, layer blocks by the mask of one side
// ---------------------------------------------------------------------------

constexpr int kDeepChildren = 24;   // child numbers of a local record (at most 20)
constexpr int kDeepLds = 160 * 1024 - 2048;   // staged children of a workgroup (beside the binomials)

// One parent of a block, by the colex rank of x's cells among the cells free
// of y: the local numbers of its children in increasing order of the new
// cell, and the mask of x's cells.
struct alignas(16) DeepLocal {
    uint16_t child[kDeepChildren];
    uint32_t mask, pad[3];
};
static_assert(sizeof(DeepLocal) == 64, "DeepLocal");

struct DeepTables {
    int e;                        // empty cells
    uint2 own, other;             // the root's stones of the mover and the other side (as PairRoot)
    uint2 slot[kDeepMaxEmpty];
    // per subset mask of the cells: its colex rank; per size, the masks by rank
    uint32_t *rank, *list;
    uint32_t list_at[kDeepMaxEmpty + 2];
    uint4 *five;                  // [2 colours: mover, other][2^e masks][2 parities of t][4 lanes]
    DeepLocal *local;             // of every layer back to back
    uint32_t local_at[kDeepMaxEmpty + 2];
};

// Everything the layers look up, one thread per (colour, mask) and per local
// parent of every layer.
__global__ void __launch_bounds__(256) deep_tables_kernel(DeepTables D, DevTables T)
{
    __shared__ BinomRow sb[kDeepMaxEmpty + 2];
    const BinomRow *bn = lds_binom(sb);
    const uint32_t masks = 1u << D.e, it = blockIdx.x * blockDim.x + threadIdx.x;
    if (it < 2 * masks) {
        const bool mine = it < masks;
        const uint32_t m = mine ? it : it - masks;
        const int size = __popc(m);
        if (mine) {
            const uint32_t r = colex_rank(m, bn);
            D.rank[m] = r;
            D.list[D.list_at[size] + r] = m;
        }
        // the mover holds at most ceil(e/2) of the cells, the other side floor(e/2)
        if (size > (mine ? (D.e + 1) >> 1 : D.e >> 1)) return;
        uint32_t lo = mine ? D.own.x : D.other.x, hi = mine ? D.own.y : D.other.y;
        for (int sl = 0; sl < D.e; sl++) {
            const uint32_t on = 0u - ((m >> sl) & 1u);
            lo |= D.slot[sl].x & on;
            hi |= D.slot[sl].y & on;
        }
        const Set256 F = five_set<SplitBits>(T.lm[lo & 511u], T.lm[512 + (lo >> 9)], T.lm[1024 + (hi & 511u)],
                                             T.lm[1536 + (hi >> 9)]);
        uint4 *dst = D.five + 8 * (size_t)it;
#pragma unroll
        for (int q = 0; q < 4; q++) {
            uint32_t even[4], odd[4];
            const uint32_t w0 = F.w[(q & 1) + 4 * (q >> 1)], w1 = F.w[(q & 1) + 4 * (q >> 1) + 2];  // p3 = 0, 1
#pragma unroll
            for (int k = 0; k < 4; k++) {
                const uint32_t u = (k & 2) ? bfi(0x0f0f0f0fu, w0 >> 4, w1) : bfi(0x0f0f0f0fu, w0, w1 << 4);
                const uint32_t z = (k & 1) ? bfi(0x33333333u, u >> 2, u) : bfi(0xccccccccu, u << 2, u);
                const uint32_t y = swap_bit0(z);
                // s = p0 where p1 + p2 + p3 + t is even
                const uint32_t zy = bfi(0x0f0f0f0fu, z, y), yz = bfi(0x0f0f0f0fu, y, z);
                const bool flip = ((k ^ (k >> 1)) & 1) != 0;
                even[k] = flip ? yz : zy;
                odd[k] = flip ? zy : yz;
            }
            dst[q] = make_uint4(even[0], even[1], even[2], even[3]);
            dst[4 + q] = make_uint4(odd[0], odd[1], odd[2], odd[3]);
        }
        return;
    }
    const uint32_t i = it - 2 * masks;
    if (i >= D.local_at[D.e + 1]) return;
    int t = 0;
    while (i >= D.local_at[t + 1]) t++;
    const int x = (t & 1) ? t >> 1 : (t + 1) >> 1, y = t - x, free_cells = D.e - y;
    DeepLocal L;
    L.mask = colex_unrank(i - D.local_at[t], x, free_cells, bn);
    L.pad[0] = L.pad[1] = L.pad[2] = 0;
    uint32_t *dst = (uint32_t *)(D.local + i);
    uint32_t word = 0, last = 0;
    int n = 0;
    for (int c = 0; c < free_cells; c++) {
        if ((L.mask >> c) & 1) continue;
        last = colex_rank(L.mask | (1u << c), bn);
        if (n & 1) dst[n >> 1] = word | (last << 16);
        else word = last;
        n++;
    }
    // the numbers up to a multiple of four repeat the last child
    for (; n & 3; n++) {
        if (n & 1) dst[n >> 1] = word | (last << 16);
        else word = last;
    }
    dst[12] = L.mask;
}

struct DeepLayer {
    const uint32_t *rank, *ylist;
    const uint4 *fx, *fy;         // five-sets of the two sides (by mask)
    const DeepLocal *local;
    const uint4 *prev;
    uint4 *cur;
    uint4 *out;
    int e, t;
    int sy;                       // stones in the cells of the side that does not move (sx: of the one that does)
    uint32_t parents, children;   // nodes of a block, of a child block
    uint32_t inner;               // layer t - 1 reads this layer in blocks of x masks: C(e - sx, sy) nodes each
    uint32_t blocks, per_group;   // blocks of the layer, blocks of a workgroup
    uint32_t parts;               // workgroups a block is split over (1 if its children are staged)
};

// ~fo & rmin(u) of a quad's node (layout above): dimension 0 flips p0, which
// s implies, dimension 3 exchanges the two p3 of a word.
__device__ __forceinline__ void deep_record(uint32_t (&r)[4], const uint32_t (&u)[4], const uint32_t (&fo)[4])
{
    uint32_t y2[4], y3[4];
#pragma unroll
    for (int k = 0; k < 4; k++) {
        y2[k] = and_quad<1>(u[k]);
        const uint32_t v = and_quad<2>(u[k]);
        y3[k] = bfi(0x0f0f0f0fu, v >> 4, v << 4);
    }
#pragma unroll
    for (int k = 0; k < 4; k++) {
        const uint32_t a = u[k], b = u[k ^ 1];
        const uint32_t ah = rotr32(a, 16), bh = (uint32_t)__builtin_amdgcn_perm(b, b, 0x02030001u);
        r[k] = andn3(fo[k], and3(a, ah, y2[k ^ 2]), and3(b, bh, y3[k]));
    }
}

__device__ __forceinline__ void unpack4(uint32_t (&w)[4], const uint4 v)
{
    w[0] = v.x; w[1] = v.y; w[2] = v.z; w[3] = v.w;
}

// One layer.  A workgroup takes per_group blocks: it copies their children,
// which lie one after another, into LDS, and its waves take 16 nodes of one
// block at a time from there.  18 empty cells: 5.47 -> 3.65 ms a solve with the
// node-per-thread form before; 12.5 GB of HBM traffic in place of 28 (11.1 GB
// are the records written and read once), VALU issue at 0.47 of the peak with
// 196 instructions of a wave to 16 nodes, the rest the chain of table loads in
// front of them.  (Read from L2 by each parent instead, the blocks
// in flight on an XCD, 50 KB and more each, exceed its L2: 15.4 GB came from
// HBM for 18 empty cells, against 5.5 GB of records.)  Blocks of more than 2500
// children (19 and 20 empty cells) do not fit: STAGED = false reads them from
// memory, several workgroups to a block (19 empty cells 16.1 -> 11.6 ms, 20
// 48.6 -> 38.3 ms with the form before).
template <int NT, bool STAGED>
__global__ void __launch_bounds__(NT, 8) deep_layer_kernel(DeepLayer J)
{
    __shared__ BinomRow sb[kDeepMaxEmpty + 2];
    extern __shared__ uint4 staged[];
    const int lane = (int)(threadIdx.x & 63u), q = lane & 3;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    // workgroups reach the 8 XCDs in turn: each XCD takes a contiguous range
    // of blocks, whose results fill neighbouring halves of the same lines
    const uint32_t per8 = gridDim.x >> 3, rem8 = gridDim.x & 7u, xcd = blockIdx.x & 7u;
    const uint32_t group = xcd * per8 + min(xcd, rem8) + (blockIdx.x >> 3);
    const uint32_t first = group / J.parts * J.per_group, part = group - group / J.parts * J.parts;
    const uint32_t nblocks = min(J.per_group, J.blocks - first);
    const uint4 *from = J.prev + 4 * (size_t)first * J.children;
    const int t = J.t, nfree = J.e - t;
    if (STAGED) {
        const uint32_t n = 4 * nblocks * J.children;
        for (uint32_t i = threadIdx.x; i < n; i += NT) staged[i] = from[i];
    }
    const BinomRow *bn = lds_binom(sb);   // (its barrier covers the copy too)
    const uint32_t *flat = &bn[0][0];
    const uint32_t winner = (t & 1) ? 0xccccccccu : 0x33333333u;
    const uint32_t chunks = (J.parents + 15) >> 4;
    // the waves of a workgroup share a block, or take blocks of their own
    const uint32_t waves = NT / 64, sharing = J.per_group >= waves ? 1u : waves / J.per_group;
    const uint32_t step = sharing * J.parts;
    for (uint32_t blk = wave / sharing; blk < nblocks; blk += waves / sharing) {
        const uint32_t y = J.ylist[first + blk];
        uint32_t Fy[4], Fz[4], below[3], term[3];
        unpack4(Fy, J.fy[8 * (size_t)y + 4 * (t & 1) + q]);
        unpack4(Fz, J.fy[8 * (size_t)y + 4 * ((t + 1) & 1) + q]);
        // lane q of a quad sums the rank terms of y's cells q, q + 4, q + 8
#pragma unroll
        for (int i = 0; i < 3; i++) below[i] = term[i] = 0;
        {
            int n = 0;
            for (uint32_t m = y; m; m &= m - 1, n++) {
                const int c = __builtin_ctz(m);
                if ((n & 3) == q) {
                    const uint32_t b = (1u << c) - 1u, to = (uint32_t)(c * (kDeepMaxEmpty + 2) + n + 1);
                    if (n < 4) { below[0] = b; term[0] = to; }
                    else if (n < 8) { below[1] = b; term[1] = to; }
                    else { below[2] = b; term[2] = to; }
                }
            }
        }
        const uint4 *kids = STAGED ? staged + 4 * blk * J.children + q : from + 4 * (size_t)blk * J.children + q;
        for (uint32_t chunk = wave % sharing + sharing * part; chunk < chunks; chunk += step) {
            const uint32_t local = 16 * chunk + (uint32_t)(lane >> 2);
            const bool mine = local < J.parents;
            const DeepLocal *loc = J.local + min(local, J.parents - 1);
            uint32_t x = loc->mask;
            const uint4 k0 = ((const uint4 *)loc)[0];
            uint4 k1 = make_uint4(0, 0, 0, 0), k2 = k1;
            if (nfree > 8) k1 = ((const uint4 *)loc)[1];
            if (nfree > 16) k2 = ((const uint4 *)loc)[2];
            // x's cells among all cells: a zero at each cell of y
            for (uint32_t m = y; m; m &= m - 1) x += x & ~((m & (0u - m)) - 1u);
            const uint32_t rx = J.rank[x];
            uint32_t Fx[4], X[4], a[4];
            unpack4(Fx, J.fx[8 * (size_t)x + 4 * (t & 1) + q]);
            const uint32_t w[12] = {k0.x, k0.y, k0.z, k0.w, k1.x, k1.y, k1.z, k1.w, k2.x, k2.y, k2.z, k2.w};
            auto child = [&](int c) { return kids[4 * ((c & 1) ? w[c >> 1] >> 16 : w[c >> 1] & 0xffffu)]; };
            if (nfree == 0) {
#pragma unroll
                for (int k = 0; k < 4; k++) a[k] = winner;
            } else {
#pragma unroll
                for (int k = 0; k < 4; k++) a[k] = 0xffffffffu;
                // four children per step, their loads issued together
#pragma unroll
                for (int c = 0; c < 20; c += 4) {
                    if (c < nfree) {
                        const uint4 v0 = child(c), v1 = child(c + 1), v2 = child(c + 2), v3 = child(c + 3);
                        uint32_t c0[4], c1[4], c2[4], c3[4];
                        unpack4(c0, v0);
                        unpack4(c1, v1);
                        unpack4(c2, v2);
                        unpack4(c3, v3);
#pragma unroll
                        for (int k = 0; k < 4; k++) a[k] = and3(a[k], c0[k], and3(c1[k], c2[k], c3[k]));
                    }
                }
            }
#pragma unroll
            for (int k = 0; k < 4; k++) {
                const uint32_t g = (uint32_t)__builtin_amdgcn_bitop3_b32(Fx[k], Fy[k], winner, 0x70);  // Fx & ~(Fy & winner)
                X[k] = (uint32_t)__builtin_amdgcn_bitop3_b32(g, Fy[k], a[k], 0xf1);                    // g | ~(Fy | a)
            }
            if (t == 0) {
                // the root's sets in the words of Set256: lane w + 8 chain takes word w = h2 + 2 p3 + 4 h3
                const int ww = lane & 7, p3 = (ww >> 1) & 1, src = (ww & 1) + 2 * (ww >> 2), sh = 2 * ((lane >> 3) & 1) + 4 * p3;
                uint32_t o = 0;
#pragma unroll
                for (int k = 0; k < 4; k++) {
                    uint32_t b = ((uint32_t)__shfl((int)X[k], src, 64) >> sh) & 0x03030303u;
                    const uint32_t z = swap_bit0(b);
                    b = (((k ^ (k >> 1)) ^ p3) & 1) ? z : b;
                    o |= ((b & 0x0303u) | ((b >> 14) & 0x0c0cu)) << (4 * (k & 1) + 16 * (k >> 1));
                }
                if (lane < 16) ((uint32_t *)J.out)[lane] = o;
            } else {
                uint32_t r[4];
                deep_record(r, X, Fz);
                // y's rank among the cells free of x
                uint32_t ry = 0;
#pragma unroll
                for (int j = 0; j < 3; j++)
                    if (4 * j < J.sy) {
                        const uint32_t v = flat[term[j] - (uint32_t)(kDeepMaxEmpty + 2) * (uint32_t)__popc(x & below[j])];
                        ry += term[j] ? v : 0u;
                    }
                ry += quad_perm<0xB1>(ry);
                ry += quad_perm<0x4E>(ry);
                if (mine) J.cur[4 * ((size_t)rx * J.inner + ry) + q] = make_uint4(r[0], r[1], r[2], r[3]);
            }
        }
    }
}

static uint64_t binom_host(int n, int k)
{
    if (k < 0 || k > n) return 0;
    uint64_t r = 1;
    for (int i = 1; i <= k; i++) r = r * (uint64_t)(n - k + i) / (uint64_t)i;
    return r;
}

static size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

static uint64_t deep_layer_nodes(int e, int t) { return binom_host(e, t) * binom_host(t, (t + 1) / 2); }

static uint64_t deep_max_layer(int e)
{
    uint64_t layer = 0;
    for (int t = 0; t <= e; t++) layer = std::max(layer, deep_layer_nodes(e, t));
    return layer;
}

// Stones in the cells of the side to move at layer t.
static int deep_movers(int t) { return (t & 1) ? t / 2 : (t + 1) / 2; }

// The scratch of the whole-table solver: offsets of its parts and total bytes.
struct DeepPlan {
    size_t rec[2], rank, list, five, local, bytes;
    uint32_t list_at[kDeepMaxEmpty + 2], local_at[kDeepMaxEmpty + 2];
};

static DeepPlan deep_plan(int e)
{
    DeepPlan P;
    memset(&P, 0, sizeof(P));
    const size_t layer = align256((size_t)deep_max_layer(e) * 64), masks = (size_t)1 << e;
    P.rec[1] = layer;
    P.rank = 2 * layer;
    P.list = align256(P.rank + 4 * masks);
    P.five = align256(P.list + 4 * masks);
    P.local = align256(P.five + 2 * masks * 128);
    for (int s = 0; s <= e; s++) P.list_at[s + 1] = P.list_at[s] + (uint32_t)binom_host(e, s);
    for (int t = 0; t <= e; t++) {
        const int sx = deep_movers(t), sy = t - sx;
        P.local_at[t + 1] = P.local_at[t] + (uint32_t)binom_host(e - sy, sx);
    }
    P.bytes = align256(P.local + (size_t)P.local_at[e + 1] * sizeof(DeepLocal));
    return P;
}

// Device bytes the deep solver needs for a root with e empty cells: two
// layers of records (64 B, or 32 B when halved by parity) and its tables.
size_t deep_scratch_bytes(int e, bool half)
{
    if (!half) return deep_plan(e).bytes;
    uint64_t sub = 0;
    for (int t = 0; t <= e; t++) sub = std::max(sub, binom_host(e, (t + 1) / 2) + binom_host(e, t / 2));
    return 2 * (size_t)deep_max_layer(e) * 32 + (size_t)sub * 32 + 256;
}

// The whole-table solve: one launch for the tables, one per layer.
static hipError_t launch_deep(int e, const unsigned cm0[4], const unsigned om0[4], const int *slot_q,
                              const int *slot_l, char *base, uint4 *out, const DevTables &T, hipStream_t st)
{
    const DeepPlan P = deep_plan(e);
    DeepTables D;
    memset(&D, 0, sizeof(D));
    D.e = e;
    D.own = make_uint2(cm0[0] | (cm0[1] << 9), cm0[2] | (cm0[3] << 9));
    D.other = make_uint2(om0[0] | (om0[1] << 9), om0[2] | (om0[3] << 9));
    for (int i = 0; i < e; i++) {
        const unsigned bit = 1u << (slot_l[i] + 9 * (slot_q[i] & 1));
        D.slot[i] = slot_q[i] < 2 ? make_uint2(bit, 0u) : make_uint2(0u, bit);
    }
    D.rank = (uint32_t *)(base + P.rank);
    D.list = (uint32_t *)(base + P.list);
    D.five = (uint4 *)(base + P.five);
    D.local = (DeepLocal *)(base + P.local);
    memcpy(D.list_at, P.list_at, sizeof(D.list_at));
    memcpy(D.local_at, P.local_at, sizeof(D.local_at));
    const uint32_t masks = 1u << e, items = 2 * masks + P.local_at[e + 1];
    hipLaunchKernelGGL(deep_tables_kernel, dim3((items + 255) / 256), dim3(256), 0, st, D, T);
    hipError_t err = hipGetLastError();
    int cur = 0;
    for (int t = e; t >= 0 && err == hipSuccess; t--, cur ^= 1) {
        DeepLayer J;
        memset(&J, 0, sizeof(J));
        J.e = e;
        J.t = t;
        const int sx = deep_movers(t);
        J.sy = t - sx;
        J.parents = (uint32_t)binom_host(e - J.sy, sx);
        J.children = (uint32_t)binom_host(e - J.sy, sx + 1);
        J.inner = (uint32_t)binom_host(e - sx, J.sy);
        J.blocks = (uint32_t)binom_host(e, J.sy);
        // at least 16 waves' worth of nodes to a workgroup, as far as LDS goes
        const bool big = (size_t)J.children * 64 > 49152;
        const uint32_t nt = big ? 1024 : 512, chunks = (J.parents + 15) / 16;
        const bool fits = (size_t)J.children * 64 <= (size_t)kDeepLds;
        J.per_group = 1;
        J.parts = 1;
        if (!fits) J.parts = std::max<uint32_t>(1, chunks / 64);
        else while (J.per_group * chunks < 16 && (size_t)(2 * J.per_group) * J.children * 64 <= 49152) J.per_group *= 2;
        J.rank = D.rank;
        J.ylist = D.list + P.list_at[J.sy];
        // the side to move is the root's mover at even layers
        J.fx = D.five + ((t & 1) ? 8 * (size_t)masks : 0);
        J.fy = D.five + ((t & 1) ? 0 : 8 * (size_t)masks);
        J.local = D.local + P.local_at[t];
        J.prev = (const uint4 *)(base + P.rec[cur ^ 1]);
        J.cur = (uint4 *)(base + P.rec[cur]);
        J.out = out;
        const uint32_t groups = (J.blocks + J.per_group - 1) / J.per_group * J.parts;
        const int lds = fits ? (int)(J.per_group * J.children * 64) : 0;
        const void *kernel = !fits ? (const void *)deep_layer_kernel<1024, false>
                           : big   ? (const void *)deep_layer_kernel<1024, true>
                                   : (const void *)deep_layer_kernel<512, true>;
        // (the same bound from every thread: another's launch may lie between)
        if (lds > 65536) err = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, kDeepLds);
        if (err != hipSuccess) break;
        void *args[] = {&J};
        err = hipLaunchKernel(kernel, dim3(groups), dim3(nt), args, (size_t)lds, st);
    }
    return err;
}

}  // namespace pg

namespace pg {

// Empty cells of a board (-1 for an invalid code).
int board_empties(uint64_t packed)
{
    int e = 0;
    for (int j = 0; j < 4; j++) {
        int x = (int)((packed >> (16 * j)) & 0xffff);
        if (x >= 19683) return -1;
        for (int l = 0; l < 9; l++, x /= 3) e += x % 3 == 0;
    }
    return e;
}

// Enqueue the deep solve of one board (packed quadrant codes) on st.
int eval_deep_enqueue(uint64_t packed, uint4 *out, hipStream_t st, int parity)
{
    if (parity < -1 || parity > 1) return fail(PENTAGO_EINVAL, "parity must be 0 or 1");
    pentago_board board;
    for (int j = 0; j < 4; j++) board.q[j] = (uint16_t)((packed >> (16 * j)) & 0xffff);
    DevTables T;
    int rc = device_tables(&T);
    if (rc) return rc;
    DeepJob J;
    memset(&J, 0, sizeof(J));
    int nb = 0, nw = 0, e = 0;
    unsigned bm[4], wm[4];
    for (int j = 0; j < 4; j++) {
        if (board.q[j] >= 19683) return fail(PENTAGO_EINVAL, "invalid quadrant code");
        bm[j] = wm[j] = 0;
        int x = board.q[j];
        for (int l = 0; l < 9; l++, x /= 3) {
            if (x % 3 == 1) bm[j] |= 1u << l;
            if (x % 3 == 2) wm[j] |= 1u << l;
        }
        nb += __builtin_popcount(bm[j]);
        nw += __builtin_popcount(wm[j]);
        for (int l = 0; l < 9; l++)
            if (!(((bm[j] | wm[j]) >> l) & 1)) {
                if (e < kDeepMaxEmpty) {
                    J.slot_q[e] = j;
                    J.slot_l[e] = l;
                }
                e++;
            }
    }
    if (nb != nw && nb != nw + 1) return fail(PENTAGO_EINVAL, "invalid stone counts");
    if (e > kDeepMaxEmpty) return fail(PENTAGO_ERANGE, "more than 20 empty cells");
    J.e = e;
    J.mover = nb == nw ? 1 : 2;
    J.parity = parity;
    const bool half = parity >= 0;
    const size_t rec = 32;  // a record of one parity
    for (int j = 0; j < 4; j++) {
        J.cm0[j] = J.mover == 1 ? bm[j] : wm[j];
        J.om0[j] = J.mover == 1 ? wm[j] : bm[j];
    }
    int dev = 0;
    hipError_t err = hipGetDevice(&dev);
    if (err != hipSuccess) return hip_fail(err, "hipGetDevice");
    {
        // the binomial table, once per device
        static std::mutex mu;
        static std::set<int> ready;
        std::lock_guard<std::mutex> lock(mu);
        if (!ready.count(dev)) {
            uint32_t tab[kDeepMaxEmpty + 2][kDeepMaxEmpty + 2];
            for (int n = 0; n < kDeepMaxEmpty + 2; n++)
                for (int k = 0; k < kDeepMaxEmpty + 2; k++) tab[n][k] = (uint32_t)binom_host(n, k);
            err = hipMemcpyToSymbol(HIP_SYMBOL(c_binom), tab, sizeof(tab));
            if (err != hipSuccess) return hip_fail(err, "binomial table upload");
            ready.insert(dev);
        }
    }
    keep_pool(dev);
    const uint64_t maxlayer = deep_max_layer(e);
    char *base = nullptr;
    err = hipMallocAsync((void **)&base, deep_scratch_bytes(e, half), st);
    if (err != hipSuccess) return hip_fail(err, "hipMallocAsync(deep scratch)");
    if (!half) {
        err = launch_deep(e, J.cm0, J.om0, J.slot_q, J.slot_l, base, out, T, st);
        (void)hipFreeAsync(base, st);
        if (err != hipSuccess) return hip_fail(err, "deep endgame launch");
        return 0;
    }
    uint4 *buf[2] = {(uint4 *)base, (uint4 *)(base + (size_t)maxlayer * rec)};
    J.ftab = (uint4 *)(base + 2 * (size_t)maxlayer * rec);
    J.out = out;
    int cur = 0;
    for (int t = e; t >= 0 && err == hipSuccess; t--) {
        J.t = t;
        J.nsub_c = (uint32_t)binom_host(e, (t + 1) / 2);
        J.nsub_o = (uint32_t)binom_host(e, t / 2);
        J.nodes = (uint32_t)(binom_host(e, t) * binom_host(t, (t + 1) / 2));
        J.cur = buf[cur];
        J.prev = buf[cur ^ 1];
        const uint32_t nsub = J.nsub_c + J.nsub_o;
        hipLaunchKernelGGL(deep_five_kernel, dim3((nsub + 255) / 256), dim3(256), 0, st, J, T);
        err = hipGetLastError();
        if (err != hipSuccess) break;
        hipLaunchKernelGGL(deep_half_kernel, dim3((J.nodes + 255) / 256), dim3(256), 0, st, J, T);
        err = hipGetLastError();
        cur ^= 1;
    }
    (void)hipFreeAsync(base, st);
    if (err != hipSuccess) return hip_fail(err, "deep endgame launch");
    return 0;
}

}  // namespace pg

using namespace pg;

extern "C" int pentago_eval_deep(pentago_board board, pentago_superinfo *out, void *hip_stream)
{
    if (!out) return fail(PENTAGO_EINVAL, "out is NULL");
    const uint64_t packed = (uint64_t)board.q[0] | ((uint64_t)board.q[1] << 16) | ((uint64_t)board.q[2] << 32) |
                            ((uint64_t)board.q[3] << 48);
    return eval_deep_enqueue(packed, (uint4 *)out, (hipStream_t)hip_stream);
}

extern "C" int pentago_eval_deep_parity(pentago_board board, int parity, pentago_superinfo *out, void *hip_stream)
{
    if (!out) return fail(PENTAGO_EINVAL, "out is NULL");
    if (parity != 0 && parity != 1) return fail(PENTAGO_EINVAL, "parity must be 0 or 1");
    const uint64_t packed = (uint64_t)board.q[0] | ((uint64_t)board.q[1] << 16) | ((uint64_t)board.q[2] << 32) |
                            ((uint64_t)board.q[3] << 48);
    return eval_deep_enqueue(packed, (uint4 *)out, (hipStream_t)hip_stream, parity);
}
