// Internal data structures of libpase (host planning + device descriptors).
//
// Vocabulary (Sec. III-B of the paper): the vertices are visited in the order
// of GenerateSeq; position i holds vertex v_i with dependent set D(i).  The DP
// table of position i, T_i, has one entry per assignment phi of D(i); the
// entry is min over the configurations c of v_i of
//     layer cost + transfer costs to later neighbours + sum_j T_j[phi' | D(j)]
// (recurrence (4)).  Here the terms of that sum are grouped by the digits of
// phi they depend on, and the "digits" of a table are the members of its
// dependent set in the table's own memory order.
#pragma once

#include <array>
#include <cstdint>
#include <string>
#include <vector>

#include "pase.h"

namespace pase {

constexpr int kMaxDims = PASE_MAX_DIMS;
constexpr int kMaxDep = PASE_MAX_DEP;
constexpr int kMaxATerms = 4;      // per-lane row terms of the row kernel
constexpr int kMaxGTerms = 24;     // terms of the generic kernel
constexpr int kMaxContrib = 64;    // contributions to one precomputed block
constexpr uint64_t kHoistElems = 1ull << 20;   // PASE_OPT_HOIST_ELEMS default
constexpr int kMaxClassEdges = 4;  // rest-digit edges of the class fill
constexpr int kMaxClassTerms = 4;  // lookups of the class fill
constexpr int kMaxBlocks = kMaxDep + 1;
constexpr uint64_t kMaxTableEntries = (1ull << 31) - 1;
constexpr uint32_t kAssignMaxDevices = 1024;   // p bound of the device assignment

// ------------------------------------------------------------------ device descriptors
struct DevVertex {            // configuration data of one vertex (uploaded once per search)
    uint64_t ex_off;          // byte offset of its split rows (K x ndims uint8)
    uint64_t L_off;           // element offset of its layer-cost vector
    uint64_t flops;           // flops_per_point * prod(size)
    uint64_t keep_n;          // prod of the sizes of the non-contracted dims
    uint32_t K, ndims, reduce_mask;
    uint32_t factors;         // 0: split rows hold log2 of power-of-two factors and the
                              // per-configuration device byte its exponent sum; 1: both
                              // hold the factors / device count themselves (p <= 255)
    uint64_t weight_n;        // gradient term: words of the weight tensor (0: no term)
    uint32_t weight_mask;
    uint32_t halo_mask;       // halo term: loop dims with a halo (0: no term)
    uint32_t input_mask;      // halo term: loop dims indexing the input tensor
    uint32_t halo_w[kMaxDims];   // halo width per loop dim
    uint64_t halo_n[kMaxDims];   // halo term: prod of the input dims' sizes other than this one
    uint32_t bits, pad;       // argmin bits of its keys (cost << bits | configuration)
};

struct DevEdge {
    uint32_t src, dst, rank;
    uint32_t factors;         // as DevVertex::factors
    int8_t sdim[kMaxDims], ddim[kMaxDims];
    uint64_t elems;
    uint64_t sig_off;         // element offset of its split signatures: K_src, then K_dst
    uint64_t mat_off;         // volume transfer model: element offset of its K_src x K_dst matrix
    uint64_t row0;            // volume transfer model: its first matrix row among all edges' rows
    uint32_t bits, pad;       // argmin bits of the end that is eliminated first: the keys its cost enters
};

// Class table of an edge shape (the class fill below): the configurations of
// the eliminated end u (K of them) and of the other end z (Kz), grouped by
// equal split signatures.  Written on the device by k_cost_tables.
struct DevClassTab {
    uint64_t ex_u, ex_z;      // byte offsets of the two ends' split rows
    // byte offsets of the outputs: for u's configurations their place when sorted by class, the inverse
    // of that, and the first place of their class (uint16[K] each); for the other end's the class's
    // places, sorted by class (zs: ClassEntry[Kz]) and by configuration (zr: first | count << 16, uint32[Kz])
    uint64_t inv_off, perm_off, first_off, zs_off, zr_off;
    uint32_t K, Kz, ndu, ndz, rank, factors, blk0, pad;
    int8_t udim[kMaxDims], zdim[kMaxDims];
};

// Class ids of a joint fill's shape (below), from its four class tables:
// consecutive numbers for the classes that occur, so that class minima are
// small arrays, and places in class order, so that a class is a range.
// Written by k_joint_tables.
constexpr uint32_t kNoClass = 0xffff;
struct JointIdI {             // of a configuration of v_i
    uint16_t own, yplace;     // places: by class of the edge to v_j; by class of the edge to y, then of that to v_j
    uint16_t other, pad;      // its class of the edge to v_j among v_j's configurations (kNoClass: none there)
};
struct JointIdJ {             // of a configuration of v_j
    uint16_t own, other;      // its class of the edge to v_i, that class among v_i's configurations
    uint16_t y, both;         // its class of the edge to y; the lowest configuration that shares both classes
};
struct JointY {               // of a configuration of y
    uint16_t i, j;            // its class among v_i's, v_j's configurations (kNoClass: none)
    uint16_t first, count;    // places by y of v_i's configurations in those that share a class of the edge
    uint16_t pj;              // between the sides, and `both` of v_j's (kNoClass: none)
    uint16_t pad[3];
};
struct DevJointTab {
    uint64_t off_i, off_j, off_y;   // byte offsets: JointIdI[Ki], JointIdJ[Kj], JointY[Ky]
    uint64_t off_start[3];    // first places of v_i's classes to v_j, v_i's to y, v_j's to y (and the end): uint16
    uint64_t off_jown;        // uint16[Kj]: by place in v_j's order to y, `other`
    int32_t tab[4];           // class tables: i to y (-1: no edge), j to y, j to i, i to j
};

struct ClassEntry {           // one configuration z of the other end
    uint16_t first, count;    // its class's configurations of u: places [first, first + count) of the sorted order
    uint32_t z;
};

// One contribution to a precomputed block element (see Prep below).
enum ContribKind : uint32_t { kContribLayer = 0, kContribEdge = 1, kContribTable = 2 };
struct Contrib {
    uint32_t kind;
    uint32_t edge;            // kContribEdge: edge id
    uint32_t dig;             // kContribEdge: plan digit of the other endpoint
    uint32_t vi_is_src;       // kContribEdge: v_i is the edge's source
    const void *ptr;          // kContribTable: value table (key type's value form, or uint64 for
                              // caller-given edge matrices)
    uint32_t sc;              // kContribTable: element stride of v_i's configuration
    uint32_t raw_u64;         // kContribTable: 1 = plain uint64 costs (caller-given edge
                              // matrices), 0 = a DP table already in this vertex's key space
    uint32_t sd[kMaxDep];     // kContribTable: element stride per plan digit (0 = unused)
};

// A precomputed block: a key-space array over (pre digits, c, post digit)
// laid out [pre...][c][ld].  Each element is the sum of its contributions,
// multiplied by 2^bits (the low bits of a key hold the configuration index).
struct Block {
    uint64_t out_off;         // element offset in the block scratch
    uint64_t elems;           // prod(pre radices) * K * ld
    uint32_t npre;
    uint32_t pre[kMaxDep];    // plan digits, slowest first
    uint32_t prerad[kMaxDep];
    int32_t post;             // plan digit, -1 = none
    uint32_t postrad;         // its radix (columns actually filled)
    uint32_t ld;              // row pitch (>= postrad, padded columns hold 0)
    uint32_t c_begin, c_end;  // contribution range
    uint32_t rows;            // prod(pre radices)
    uint32_t chunks;          // workgroups per row: ceil(K * ld / (kPrepThreads * span))
    uint32_t wg_begin;        // first workgroup of this block
    uint32_t span;            // kPrepThreads-element spans per workgroup
};

constexpr uint32_t kPrepThreads = 256;

struct PrepArgs {
    uint32_t vi, K, bits, nblocks;
    uint64_t total;           // sum of block elements
    uint32_t nwg, pad;        // workgroups of this vertex
    void *blocks;             // this vertex's block scratch
    Block blk[kMaxBlocks];
};

// One vertex of a batched launch: its descriptor index and its first
// workgroup.  The workgroups of a launch are the concatenation
// of the workgroups of its vertices.
struct BatchEntry {
    uint32_t pos;             // sequence position (host)
    uint32_t idx;             // its descriptor of the launch's kind
    uint32_t first;
    uint32_t prio;            // 1: the bulk lane schedule's small vertices -- their waves issue first
    uint32_t kind;            // row-kernel launches: 0 a row fill, 1 a two-term generic fill riding along
};
constexpr uint32_t kEntryGeneric2 = 1;

struct ATerm {                // per-lane row term of the row kernel (key space)
    const void *ptr;
    uint32_t sc;              // stride of c
    uint32_t bytes;           // size of the array (buffer-load range, < 2^31)
    uint32_t sdO[kMaxDep];    // strides per outer digit
    uint32_t sdR[kMaxDep];    // strides per row digit
};

struct RowsArgs {
    const void *B;            // [o][c][ldz] key space: layer cost, c, outer and column terms
    uint32_t ldz, Kz, K, bits;
    uint32_t MO, MR, tiles_per_o, nchunks;
    uint32_t nsplit, cper;
    uint32_t nO, nR;
    uint32_t radO[kMaxDep], radR[kMaxDep];
    uint32_t na;
    ATerm a[kMaxATerms];
    void *T;                  // output values, index z*(MO*MR) + o*MR + r
    uint16_t *A;              // output argmins
    void *partial;            // nsplit > 1: keys [split][N]
    uint64_t N;
    uint64_t total_tiles;     // tiles (a workgroup takes 4 / parts of them)
    uint32_t nblocks_launched;
    uint32_t parts;           // waves sharing one tile's c range: 1, 2 or 4
    uint32_t out_shift;       // bits of the table's reader: values are stored x 2^out_shift
    // Fused minimum of the reader (fz_keys non-null): the table's only reader
    // v_j is this vertex's column digit and takes, per row r, the minimum over
    // its configuration c = z of T[z][r] plus its other row terms at (r, z)
    // plus its column block at z.  The epilogue forms those keys of v_j for
    // the tile's columns and min-combines them into fz_keys[r] atomically (64-bit
    // keys, non-negative, so their bit patterns order like the keys); a
    // one-split reduction then turns the keys into v_j's table.  T may then
    // be null: nothing else reads it.
    void *fz_keys;
    const void *fz_B;         // the reader's column block, element z * fz_ldz
    uint32_t fz_ldz, fz_na;   // its row pitch; the reader's row terms other than T
    ATerm fz_a[kMaxATerms];   // those row terms (ptr, sc, sdR over the same row digits)
};

struct GTerm {                // term of the generic kernel (key space)
    const void *ptr;
    uint32_t sc, pad;
    uint32_t sd[kMaxDep];
};

struct GenericArgs {
    uint32_t m, K, bits, nt;
    uint32_t group_log2;      // lanes per entry = 2^group_log2 (c is strided over them)
    uint32_t pad2;
    uint32_t rad[kMaxDep];    // radices of the plan digits (= T_i layout), slowest first
    GTerm t[kMaxGTerms];
    void *T;
    uint16_t *A;
    uint64_t N;
    uint32_t out_shift, nblk;  // nblk: workgroups of this vertex
};

// Direct fill of a small vertex: every term of recurrence (4) -- layer cost,
// transfer costs, table lookups -- is summed per (entry, c) from its source
// arrays (contributions [c_begin, c_end) over the plan digits), with no prep
// blocks; one launch per level instead of prep + fill (+ split reduction).
struct DirectArgs {
    uint32_t vi, K, bits, out_shift;
    uint32_t m;               // plan digits (= T_i layout), slowest first
    uint32_t group_log2;      // lanes per entry = 2^group_log2 <= 256 (c is strided over them)
    uint32_t c_begin, c_end;  // contributions
    uint32_t rad[kMaxDep];
    uint32_t nblk, pad;       // nblk: workgroups of this vertex
    uint64_t N;
    void *T;
    uint16_t *A;
};

// Class fill.  With the split match model an edge's cost is
//     r * t_x(c, z) = 0 if c and z split the tensor alike (one class), else min(f(c), f(z)),
//     f(x) = r * ceil(elems / P_x)
// (the larger device count gives the smaller cost), and 0 <= f, so for a digit
// z that meets v_i in this one edge and in no lookup, with X[c][rest] the sum
// of all other terms,
//     min_c X[c] + t_x(c, z) = min( min_{c in class of z} X[c],  f(z) + min_c X[c],  min_c (X[c] + f(c)) ):
// K * rest evaluations of X and about two minima per table entry instead of K
// adds and minima per entry.  Every term on the right is a key of a
// configuration or an upper bound of one, so minimum and argmin are those of
// the left.  Without such a digit (has_z = 0) the fill is the minimum over c
// of X itself.
struct ClassEdge {            // an edge to a rest digit
    const uint64_t *sig_c, *sig_o;   // split signatures by c, by the other end's configuration
    const void *f_c, *f_o;           // f of the two ends, key space
    uint32_t dig, pad;               // rest digit of the other end
};

struct ClassTerm {            // a lookup T_j (key space)
    const void *ptr;
    uint32_t sc, raw;         // element stride of c; 1: plain uint64 costs (a volume model edge's matrix)
    uint32_t sd[kMaxDep];     // element strides of the rest digits
};

struct ClassArgs {
    const void *Lk;           // key-space layer costs: (cost << bits) + c
    const uint16_t *inv;      // class table of the edge to z
    const ClassEntry *zs;
    const void *fzc, *fzo;    // f of that edge by c, by z
    void *T;                  // index z * rows + row (without z: row)
    uint16_t *A;
    uint32_t K, Kz, bits, out_shift;
    uint32_t rows, nR;        // rows = product of the rest radices (slowest first)
    uint32_t rad[kMaxDep];
    uint32_t lr, has_z;       // a workgroup takes 2^lr rows
    uint32_t staged;          // many rows: per-configuration data staged through LDS
    uint32_t keep;            // staged: 1: X of all K configurations and rows in LDS; 0: lr = 6 and X formed twice
    uint32_t ne, nt, nblk, lds;   // lds: bytes of dynamic LDS
    ClassEdge e[kMaxClassEdges];
    ClassTerm t[kMaxClassTerms];
    const uint64_t *sig_zc, *sig_zo;   // signatures of the edge to z by c, by z (one entry's evaluation)
};

// Joint fill.  A vertex i without a class digit whose lookup T_j does have one
// in c: v_j meets v_i in one edge and in no lookup of its own, and a digit y of
// T_j meets v_j in one edge and no lookup, v_i in at most one edge, and no other
// lookup of i.  Then
//     T_i[rest][y] = min_{c, c'} XI[c] + XJ[c'] + t(c', c) + t_i(c, y) + t_j(c', y)
// with XI, XJ the sums of i's and j's other terms (functions of the rest
// digits only), and each t one of 0 (same class), f of one end, f of the other.
// Expanding them, with J0[c] = min_c' XJ + t, J1[c] = min_c' XJ + f_y(c') + t
// and I0, I1 alike over c, the minimum over all cases is that of
//     min_c t_i(c, y) + XI[c] + min(J0[c] + f_y'(y), J1[c]),
//     min_{c' in class of y} XJ[c'] + min(I0[c'] + f(y), I1[c'], min_{c in class of y} XI[c] + t(c', c)),
// all of which are minima over classes and over everything: per row a few
// times K_i + K_j + Kz operations instead of K_i * Kz, and T_j itself is never
// formed.  f >= 0 makes every case an upper bound of the true cost, so minimum
// and argmin are those of the dense fill.  (v_j's configuration is looked up
// in the back-substitution by one evaluation of its K_j keys.)
//
// Everything on v_j's side depends on XJ's digits alone, which are some of the
// rest digits (called upper; the others are lower): the half fill computes,
// per upper index, J0 and J1 by c and the minima of XJ and XJ + f over y's
// classes, and the joint fill combines them with XI for every lower index.
struct JointSide {            // terms of one side
    const void *Lk;           // key-space layer costs
    uint32_t K, ne, nt;
    int32_t shift;            // its keys x 2^shift are keys of v_i (0 for v_i itself)
    ClassEdge e[2];           // (digits: of the upper and lower digits together, slowest first)
    ClassTerm t[2];
};

struct JointArgs {
    JointSide s[2];           // v_i, v_j
    const void *fi_o, *fj_o;  // f of the edge between them by c, by c' (v_j's key space)
    const void *fi_y, *fi_yy; // f of the edge from v_i to y by c, by y (null: no edge)
    const void *fj_y, *fj_yy; // of the edge from v_j to y by c', by y (v_j's key space)
    const JointIdI *ii;
    const JointIdJ *ij;
    const JointY *y;
    const uint16_t *start_o, *start_yi, *start_yj, *jown;
    const uint16_t *jplace;   // v_j's places in its order to y
    // half table, per upper index: J0[Ki], J1[Ki], XJ[Kj] by place in the order to y, and by y the minima
    // of XJ, of XJ + f, of XJ over the pair's combined class (Ky each)
    void *half;
    void *T;                  // index (upper * lower count + lower) * Ky + y
    uint16_t *A;
    uint32_t Ky, bits, out_shift, has_e;   // has_e: v_i has an edge to y
    uint32_t oi, oj, yi, yj;  // classes: of the edge between the sides among v_i's, v_j's; of those to y
    uint32_t upper, lower, nR;   // table rows = upper * lower
    uint32_t rad[kMaxDep];
    uint32_t seg;             // workgroups per upper index
    uint32_t nblk, hblk, threads, lds, hlds;   // h: of the half fill
};

constexpr uint32_t kJointMaxK = 1024;         // past 768: two configurations per thread of a 512-thread workgroup
constexpr uint32_t kJointTerms = 2;           // rest edges, and lookups, per side
constexpr uint32_t kJointMaxLds = 80 << 10;   // two workgroups per CU
inline uint64_t joint_half_elems(uint64_t Ki, uint64_t Kj, uint64_t Ky) { return 2 * Ki + Kj + 3 * Ky; }
inline uint64_t joint_lds(uint64_t Ki, uint64_t Kj, uint64_t oi, uint64_t yi, uint64_t yj, bool has_e) {
    return 8 * (32 + Ki + oi + yj + Kj + (has_e ? 6 * Ki + oi + 4 * yi + yj : 0)) + 2 * (oi + yi + yj + 3 + Kj) + 16;
}
inline uint64_t half_lds(uint64_t Kj, uint64_t oj, uint64_t yj) { return 8 * (16 + 2 * oj + 2 * yj + Kj); }

// Exchange fill.  A pair (j, i) where j has no edges and three lookups
// of one digit each -- A over v_i, B over y, C over z -- and i, with an edge
// to y and one to z, reads T_j alone:
//     T_i[y][z] = min_x L_i[x] + t1(x, y) + t2(x, z) + min_c L_j[c] + A[c][x] + B[c][y] + C[c][z].
// With the minima exchanged the inner one, over x at a fixed c, is that of
// A'[x] = A[c][x] + L_i[x] plus two split-match edges, each of which is 0
// (same class), f of x or f of the other end: minima of A' over everything, a
// class of y, a class of z, or both.  So per c a few arrays over y and over z
// (the half table), and
//     T_i[y][z] = min_c min( a1[c][y] + C[c][z] + f2(z),  b1[c][y] + C[c][z],
//                            B[c][y] + g[c][z] + f1(y),   B[c][y] + d[c][z],
//                            B[c][y] + C[c][z] + I[c][x both classes] ):
// about ten operations per (c, y, z) instead of two per (c, x, y, z), and T_j
// is never formed.  Every case is a key of some x or an upper bound of one, so
// minimum and lowest argmin are those of the two dense fills; j's argmin is
// evaluated in the back-substitution.
struct ExchLookup {           // one-digit lookup of v_j
    const void *ptr;
    uint32_t sc, sd;          // element strides of c and of the digit
};

struct ExchArgs {
    const void *Li, *Lj;      // key-space layer costs
    ExchLookup l[3];          // over x = v_i, y, z (v_j's key space)
    const void *f1x, *f1y, *f2x, *f2z;   // f of the edges to y and z, by x and by the other end (v_i's)
    // class tables of x by the edges to y and z
    const uint16_t *perm1, *first1, *first2;
    const uint32_t *zr1, *zr2;
    // per c: a1, b1 and B by y (Kyp each), C, g and d by z, I by x
    void *half;
    void *T;                  // index y * Kz + z
    uint16_t *A;
    uint32_t Ki, Kj, Ky, Kyp, Kz;   // Kyp: Ky rounded up to kExchCols
    int32_t shift;            // v_j's keys x 2^shift are v_i's
    uint32_t bits, out_shift;
    uint32_t nblk, lds;       // workgroups of the fill; dynamic LDS of the half fill
};

constexpr uint32_t kExchCols = 4;             // y's per workgroup of the fill (one per wave in its last step)
constexpr uint32_t kExchMaxK = 1024;          // v_i's configurations (48 bytes of LDS each)
inline uint64_t exch_half_elems(uint64_t Ki, uint64_t Kj, uint64_t Kyp, uint64_t Kz) { return Kj * (3 * Kyp + 3 * Kz + Ki); }
inline uint64_t exch_lds(uint64_t Ki) { return 8 * (4 + 5 * Ki) + 6 * Ki + 16; }

constexpr uint32_t kClassMaxK = 4096;         // configurations of either end of the class edge
constexpr uint32_t kClassMaxLds = 64 << 10;   // two workgroups per CU (160 KB) with room beside them
constexpr uint32_t kClassTabLanes = 16;       // threads per configuration of the class tables' counting
constexpr uint32_t kClassStagedRows = 4;      // log2 of the rows per workgroup from which data is staged
// dynamic LDS of one workgroup: per-wave minima and X; staged: also the per-configuration records, the
// class entries and the configurations of the lookups
inline uint64_t class_lds(uint64_t K, uint64_t Kz, uint32_t ne, uint32_t nt, uint32_t lr, bool has_z, bool keep,
                          uint32_t threads) {
    const uint64_t red = (threads / 64) * (16ull << (lr < 6 ? lr : 6)), x = keep ? (K << lr) * 8 : 0;
    if (lr < kClassStagedRows) return red + x;
    return red + x + K * (16 + 16 * ne + (nt ? 4 : 0)) + (has_z ? Kz * 16 : 0);
}

struct ReduceArgs {
    const void *partial;
    void *T;
    uint16_t *A;
    uint64_t N;
    uint32_t nsplit, bits, out_shift, nblk;
};

struct BacktrackDesc {        // per position, for the back-substitution kernel
    const uint16_t *A;
    uint32_t vi, m;
    uint32_t level;           // backward level: 1 + max level over D(i) (0 when D(i) is empty)
    uint32_t K;               // configurations of v_i: a stored argmin must be below it
    uint32_t dig[kMaxDep];    // vertex ids of the layout digits
    uint64_t stride[kMaxDep];
    const ClassArgs *lazy;    // table not formed (the vertex is part of a joint fill): its terms; else null
    uint32_t pos, pad;
};

constexpr uint32_t kMaxBacktrackThreads = 1024;   // one thread per position

struct SearchOut {            // written by the back-substitution kernel
    uint64_t min_cost;
    uint32_t status;          // 0 = ok; 4 = an argmin out of range
    uint32_t pad;
};

// PASE_OPT_SCHEDULE values
enum SchedKind { kSchedLevel = 0, kSchedSeq = 1, kSchedBulk = 4, kSchedSplit = 5 };
constexpr int kSplitBatchedLevels = 1;   // split chains: levels that stay batched on one lane

// ------------------------------------------------------------------ host plan
struct TermRef {
    int j;                    // position of the producer (last vertex of the component)
    std::vector<int> dig;     // D(j) - {v_i}: vertex ids
};

// Kinds of launch descriptors: a vertex has those its launches need.
enum DescKind { kDescPrep, kDescRows, kDescGeneric, kDescReduce, kDescDirect, kDescClass, kDescJoint, kDescExch, kDescKinds };

// bytes of one descriptor of each kind
constexpr uint64_t kDescBytes[kDescKinds] = {sizeof(PrepArgs), sizeof(RowsArgs), sizeof(GenericArgs), sizeof(ReduceArgs),
                                             sizeof(DirectArgs), sizeof(ClassArgs), sizeof(JointArgs), sizeof(ExchArgs)};

enum KernelKind { kGeneric = 0, kRows = 1, kDirect = 2 };

struct VPlan {
    int vi = -1;
    uint32_t K = 0, bits = 0;
    std::vector<int> D;             // D(i), ascending vertex id
    std::vector<int> layout;        // plan digits = T_i memory order, slowest first (vertex ids)
    std::vector<uint64_t> stride;   // element stride of each layout digit in T_i
    uint64_t N = 1;
    std::vector<int> edges;         // edges joining v_i and a later vertex
    std::vector<TermRef> terms;     // one lookup per connected subset in S(i)
    int consumer = -1;              // position whose lookups read T_i
    uint32_t out_shift = 0;         // T_i is stored x 2^(bits of its reader): in the reader's key space
    KernelKind kernel = kGeneric;
    // row kernel shape
    int z = -1;                     // column digit (vertex id)
    // class fill (kernel kRows or kDirect): z is then the class digit (-1: none), R the rest
    // digits, and every term is read from its source array (no prep blocks)
    bool classes = false;
    uint32_t lr = 0;                // log2 of the rows per workgroup
    bool keep = false;              // X kept in LDS
    uint32_t threads = 256;         // workgroup size
    int ctab = -1;                  // its class table
    // joint fill (kernel kRows): position of the vertex whose table it does without (-1: none), with z
    // the digit y, R the rest digits, and four class tables (i to y, j to y, j to i, i to j)
    int joint = -1;
    int jtab[4] = {-1, -1, -1, -1};
    // exchange fill: joint names the other vertex as well; the first two of jtab are v_i to y and to z, the
    // plan digits
    bool exch = false;
    int jshape = -1;                // its class ids
    uint32_t jcls[4] = {0, 0, 0, 0};   // classes: i and j to y, j to i, i to j
    uint64_t jupper = 1;            // product of the upper digits (the first of R)
    bool jearly = false;            // the half fill runs in the other vertex's slot, else just before the fill
    int absorbed = -1;              // the vertex whose joint fill does without this one's table
    uint32_t desc[kDescKinds] = {}; // index of its descriptor of each kind
    std::vector<int> O, R;          // outer / row digits (vertex ids), slowest first
    uint32_t TZ = 0, TM = 1, ldz = 0, nchunks = 0, nsplit = 1, cper = 0, parts = 1;
    uint64_t MO = 1, MR = 1;
    uint32_t na = 0;                // row kernel: per-lane row terms
    // fused minimum (row kernel): this vertex's table feeds only the minimum
    // of its column digit's vertex, which its fill forms in the epilogue
    int fuse_into = -1;             // position of that reader, -1 = none
    int fused_from = -1;            // the reader: position of the producer, -1 = none
    uint64_t fkeys_off = 0;         // the reader: bytes into the fused-key region
    // hoisted prep: the blocks read only tables filled by slot prep_after or
    // earlier, so they are built right after that slot, beside the slots in
    // between -- on a side stream (level layout), or at the end of that
    // slot's group of lane prep_lane (lanes); -2 = not hoisted
    int prep_after = -2;
    int prep_lane = 0;
    double fill_ms = 0;             // last profiled fill time
    double est_us = 0;              // planned fill time (tile model), for the schedule
    // memory
    uint64_t T_off = 0, A_off = 0;  // bytes into the table arenas
    uint64_t block_elems = 0;       // block scratch this vertex needs
    uint64_t block_off = 0;         // bytes into the block scratch
    uint64_t partial_off = 0;       // bytes into the split scratch
    // schedule
    int level = 0;                  // dependency level: 1 + max level of the tables it reads
    int slot = 0;                   // launch slot: its level (level schedule) or its position
    int lane = 0;                   // lane schedules: 0 = the side stream (small vertices, level by level),
                                    // 1 = the caller's stream (the leaves, the large fills and their readers)
};

struct Plan {
    std::vector<int> seq, pos;
    std::vector<VPlan> v;           // by position
    uint64_t cells = 0, entries = 0, rows_cells = 0, stream_cells = 0;
    uint32_t max_dep = 0, rows_vertices = 0;
    // upper bounds per position (cost_bounds), of the current costs; bounds: -1 not evaluated, 0 past 64 bits, 1 valid
    int bounds = -1;
    std::vector<uint64_t> qmax, tmax;
    // workspace layout, byte offsets from the workspace base
    uint64_t off_ex = 0, off_vert = 0, off_edge = 0, off_L = 0, off_lsum = 0, off_sig = 0,
             off_ovedge = 0, off_contrib = 0,
             off_bt = 0, off_zero = 0, off_cfg = 0, off_out = 0, off_vmat = 0, off_T = 0, off_A = 0, off_block = 0,
             off_partial = 0, off_fused = 0, total = 0;
    uint64_t T_bytes = 0, A_bytes = 0, block_bytes = 0, partial_bytes = 0, contrib_count = 0;
    uint64_t fused_bytes = 0;       // keys of the fused minima (initialised by k_cost_tables)
    uint32_t hoisted = 0;           // vertices whose prep runs on the side stream
    uint32_t fused = 0;             // fused producer/reader pairs
    uint64_t sig_count = 0;         // split signatures of all edge endpoints
    int nslots = 0;                 // launch slots (levels, or positions when sequential)
    bool by_level = false;          // the vertices of one dependency level share launches
    bool resident = false;          // every table and scratch buffer resident at once (no reuse)
    uint64_t off_desc[kDescKinds] = {}, off_batch = 0;   // launch descriptors by kind, batch tables
    uint32_t ndesc[kDescKinds] = {};
    // class fills: tables per edge shape (byte offsets relative to off_ctab until layout) and the
    // key-space layer costs and edge f values, all written by k_cost_tables
    std::vector<DevClassTab> ctabs;
    std::vector<DevJointTab> jtabs;
    uint32_t class_fills = 0, joint_fills = 0, ctab_blocks = 0;
    uint64_t off_ctdesc = 0, off_jtdesc = 0, off_ctab = 0, off_Lk = 0, off_fk = 0;
    bool overridden = false;        // planned for caller-given costs
};

// Positions whose tables the launches of a vertex read: a joint fill's half
// fill runs in the other vertex's slot (its tables are that vertex's reads),
// or, without levels or hoisting, just before the fill.
template <typename F> void for_reads(const Plan &P, const VPlan &vp, F f) {
    for (const auto &t : vp.terms) {
        if (t.j == vp.joint && !vp.jearly) {
            for (const auto &u : P.v[t.j].terms) f(u.j);
        } else f(t.j);
    }
}

struct DeviceState;   // defined by the device runtime

}  // namespace pase

struct pase_graph_s {
    std::vector<pase_vertex_desc> V;
    std::vector<pase_edge_desc> E;
    uint64_t r = 8;
    uint32_t seq_rule = 0;
    std::vector<std::vector<int>> nbr;     // undirected, deduplicated, ascending
    std::string err;
    // options
    bool keep_tables = false;
    bool dense_only = false;        // no class, joint or exchange fills: they do not fit the memory at hand
    uint64_t structured_total = 0;  // dense_only: the workspace with them
    int profile = 0;                // pase_option PASE_OPT_PROFILE: 0 off, 1 every fill launch, 2 the
                                    // column-form row-kernel launches only
    uint64_t mem_budget = 64ull << 30;
    int kernel_mode = 0, key_mode = 0;
    uint32_t tile_cols = 0, tile_rows = 0, tile_parts = 0, c_splits = 0;   // 0 = chosen by the plan
    int schedule = pase::kSchedSplit;   // pase_option PASE_OPT_SCHEDULE (SchedKind)
    int order_mode = 0;             // pase_option PASE_OPT_ORDER: 0 GenerateSeq, 1 breadth-first
    // configurations
    bool enumerated = false;
    uint32_t config_set = 0;        // pase_option PASE_OPT_CONFIG_SET, read by pase_enumerate_configs
    uint32_t transfer_opt = 0;      // pase_option PASE_OPT_TRANSFER, read by pase_enumerate_configs
    uint32_t grad_opt = 0;          // pase_option PASE_OPT_GRAD_SYNC, read by pase_enumerate_configs
    uint32_t halo_opt = 0;          // pase_option PASE_OPT_HALO, read by pase_enumerate_configs
    bool halo = false;              // the enumerated layer costs carry the halo term
    std::vector<std::array<uint64_t, pase::kMaxDims>> halo_n;   // halo term: per vertex and loop dim, the
                                    // product of the input dims' sizes other than that dim
    uint64_t direct_cells = 1ull << 18;  // pase_option PASE_OPT_DIRECT_CELLS
    uint32_t bulk_us = 100;         // pase_option PASE_OPT_BULK_US
    bool fuse_min = true;           // pase_option PASE_OPT_FUSED_MIN
    uint64_t hoist_elems = pase::kHoistElems;   // pase_option PASE_OPT_HOIST_ELEMS (0 = never)
    std::vector<uint64_t> weight_n; // gradient term of the enumeration: weight words per vertex (0 = none)
    bool volume = false;            // the enumerated transfer model is the volume intersection
    std::vector<uint64_t> mat_off;  // volume model: element offset of each edge's cost matrix
    uint64_t mat_total = 0;         // volume model: entries of all edge matrices
    std::vector<uint64_t> mat_row0; // volume model: first matrix row of each edge (rows = K_src)
    uint64_t mat_rows = 0;          // volume model: rows of all edge matrices
    uint32_t p = 0;
    bool factors = false;           // the enumerated set: split rows hold factors, not exponents
    std::vector<uint32_t> K;
    // the configurations of a vertex depend only on its dimension count: one
    // row set per count, ex_rows[d][c*d + k] = log2 of the split factor, or the
    // factor itself when `factors`
    std::vector<std::vector<uint8_t>> ex_rows;
    std::vector<const std::vector<uint8_t> *> ex;  // [v] -> ex_rows[ndims of v]
    std::vector<uint64_t> flops, keep_n;
    std::vector<uint64_t> maxL;            // upper bound of the layer cost per vertex
    std::vector<uint64_t> maxR;            // upper bound of the transfer cost per edge
    // caller-given costs
    bool overridden = false;
    std::vector<uint64_t> ov_layer, ov_edge, ov_layer_off, ov_edge_off;
    // plan
    pase::Plan plan;
    bool planned = false;
    // keys of the plan (R10): 0 fp64, 1 uint64, 2 128-bit (packed keys past 2^64 while every
    // cost sum fits 64 bits; such a plan runs every vertex on prep + the generic kernel)
    uint32_t plan_key_type = 0;
    bool plan_wide = false;         // the plan was built for 128-bit keys
    // last search
    bool searched = false;
    uint32_t key_type = 0;
    pase_run_stats stats{};
    // a workspace lent by the caller (pase_set_workspace), else library-owned memory
    void *lent_ws = nullptr;
    uint64_t lent_bytes = 0;
    // device runtime
    pase::DeviceState *dev = nullptr;
};

namespace pase {
// host.cpp
pase_status fail(pase_graph_t g, pase_status st, const std::string &msg);
uint32_t choose_key_type(pase_graph_t g, pase_status *st);
uint32_t key_bytes(pase_graph_t g);   // bytes of a table value / block key of the plan (8 or 16)
// launch_plan.cpp: the launch descriptors and constant image of the plan's key
// type, built against a stand-in workspace base into a host buffer of exactly
// the constant region's size (no device work)
pase_status plan_check(pase_graph_t g, uint64_t *image_bytes);
// device.hip
void device_release(pase_graph_t g);
pase_status device_search(pase_graph_t g, void *stream, uint64_t *min_cost, uint32_t *cfg);
pase_status device_search_noalloc(pase_graph_t g, void *stream, uint64_t *min_cost, uint32_t *cfg);
pase_status device_table_entry(pase_graph_t g, int pos, uint64_t idx, uint64_t *cost,
                               uint32_t *arg);
pase_status device_fingerprint(pase_graph_t g, int pos, uint64_t *fpT, uint64_t *fpA);
pase_status device_layer_costs(pase_graph_t g, uint32_t v, uint64_t *out);
pase_status device_edge_costs(pase_graph_t g, uint32_t e, uint64_t *out);
}  // namespace pase
