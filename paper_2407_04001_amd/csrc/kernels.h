// Device code of the kernels of libpase (gfx950): key arithmetic, the device
// cost model, and the work of one workgroup of each kernel ("items").
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "internal.h"

namespace pase {

// ------------------------------------------------------------------ key arithmetic
template <typename KeyT> struct KeyOps;

// Val: the type of a stored table value (cost x 2^out_shift, in its reader's
// key space); Acc: an exact integer wide enough for one key, in which prep
// sums its contributions before the key is formed.
template <> struct KeyOps<double> {
    using Val = double;   // table value type
    using Acc = uint64_t;
    static constexpr double sentinel() { return 1152921504606846976.0; }  // 2^60 > any key
    __device__ static double from_u64(uint64_t x) { return (double)x; }
    __device__ static double from_acc(uint64_t x) { return (double)x; }
    __device__ static uint64_t val_to_u64(double x) { return (uint64_t)x; }
    __device__ static uint64_t val_to_acc(double x) { return (uint64_t)x; }
    __device__ static uint64_t unshift(double x, uint32_t s) { return (uint64_t)x >> s; }
    __device__ static double add(double a, double b) { return a + b; }
    __device__ static double min(double a, double b) { return __builtin_fmin(a, b); }
    // key = cost * 2^bits + c  ->  (cost * 2^out_shift, c)
    __device__ static void split(double key, uint32_t bits, uint32_t out_shift, double &val, uint32_t &c) {
        double s = __builtin_ldexp(1.0, (int)bits);
        double v = __builtin_trunc(key * __builtin_ldexp(1.0, -(int)bits));
        val = v * __builtin_ldexp(1.0, (int)out_shift);
        c = (uint32_t)__builtin_fma(-v, s, key);
    }
};

template <> struct KeyOps<uint64_t> {
    using Val = uint64_t;
    using Acc = uint64_t;
    static constexpr uint64_t sentinel() { return ~0ull; }
    __device__ static uint64_t from_u64(uint64_t x) { return x; }
    __device__ static uint64_t from_acc(uint64_t x) { return x; }
    __device__ static uint64_t val_to_u64(uint64_t x) { return x; }
    __device__ static uint64_t val_to_acc(uint64_t x) { return x; }
    __device__ static uint64_t unshift(uint64_t x, uint32_t s) { return x >> s; }
    __device__ static uint64_t add(uint64_t a, uint64_t b) { return a + b; }
    __device__ static uint64_t min(uint64_t a, uint64_t b) { return a < b ? a : b; }
    __device__ static void split(uint64_t key, uint32_t bits, uint32_t out_shift, uint64_t &val, uint32_t &c) {
        val = (key >> bits) << out_shift;
        c = (uint32_t)(key & ((1ull << bits) - 1));
    }
};

// 128-bit keys: cost * 2^bits + c for costs up to 2^64 (bits <= 16), so the
// packed key never overflows; table values are stored in 16 bytes.
using u128 = unsigned __int128;
template <> struct KeyOps<u128> {
    using Val = u128;
    using Acc = u128;
    static constexpr u128 sentinel() { return ~(u128)0; }
    __device__ static u128 from_acc(u128 x) { return x; }
    __device__ static uint64_t val_to_u64(u128 x) { return (uint64_t)x; }
    __device__ static u128 val_to_acc(u128 x) { return x; }
    __device__ static uint64_t unshift(u128 x, uint32_t s) { return (uint64_t)(x >> s); }
    __device__ static u128 add(u128 a, u128 b) { return a + b; }
    __device__ static u128 min(u128 a, u128 b) { return a < b ? a : b; }
    __device__ static void split(u128 key, uint32_t bits, uint32_t out_shift, u128 &val, uint32_t &c) {
        val = (key >> bits) << out_shift;
        c = (uint32_t)key & ((1u << bits) - 1u);
    }
};


// Buffer resource word 3 (data format 32-bit, raw addressing) for gfx9-family
// buffer instructions.
constexpr int kBufferWord3 = 0x00020000;

// ------------------------------------------------------------------ cost model (device)
// Layer cost t_l(v, c) = ceil(F / P) + r * (P_red - 1) * ceil(keep / (P / P_red)),
// with P the device count of the configuration and P_red the product of the
// split factors of the contracted dims.  With power-of-two factors (split rows
// hold exponents) the divisions are shifts; otherwise (rows hold the factors,
// P <= 255) they are integer divisions.  The host has bounded every operand so
// nothing overflows.
__device__ __forceinline__ uint64_t ceil_div_u64(uint64_t a, uint32_t b) { return (a + (b - 1)) / b; }

// Optional weight-gradient term: the weight tensor (weight_n words) is cut
// into shards of S = ceil(weight_n / P_w) words by the splits of its dims and
// each shard lives on the R = P / P_w devices that differ in the other dims;
// a ring all-reduce moves ceil(2 (R - 1) S / R) = 2S - floor(2S / R) words.
// Optional halo term: for every split loop dim k with a halo of width w, each
// part receives w boundary rows of the input from both neighbours along k; a
// row is the part's share of the input over its other dims:
// 2 w ceil(halo_n[k] / (product of the other input dims' splits)) words.
__device__ __forceinline__ uint64_t halo_cost(const DevVertex &dv, const uint8_t *ex, uint64_t r) {
    uint64_t words = 0;
    for (uint32_t k = 0; k < dv.ndims; k++) {
        if (!((dv.halo_mask >> k) & 1u) || ex[k] == (dv.factors ? 1 : 0)) continue;
        uint32_t S = dv.factors ? 1 : 0;
        for (uint32_t j = 0; j < dv.ndims; j++)
            if (j != k && ((dv.input_mask >> j) & 1u)) S = dv.factors ? S * ex[j] : S + ex[j];
        const uint64_t part = dv.factors ? ceil_div_u64(dv.halo_n[k], S)
                                         : (dv.halo_n[k] + ((1ull << S) - 1)) >> S;
        words += 2ull * dv.halo_w[k] * part;
    }
    return r * words;
}

__device__ __forceinline__ uint64_t layer_cost(const DevVertex &dv, const uint8_t *ex, uint64_t r) {
    const uint64_t halo = dv.halo_mask ? halo_cost(dv, ex, r) : 0;
    if (dv.factors) {
        uint32_t P = 1, red = 1, Pw = 1;
        for (uint32_t k = 0; k < dv.ndims; k++) {
            P *= ex[k];
            if ((dv.reduce_mask >> k) & 1u) red *= ex[k];
            if ((dv.weight_mask >> k) & 1u) Pw *= ex[k];
        }
        uint64_t cost = ceil_div_u64(dv.flops, P) + r * ((uint64_t)(red - 1) * ceil_div_u64(dv.keep_n, P / red));
        if (dv.weight_n) {
            const uint64_t S2 = 2 * ceil_div_u64(dv.weight_n, Pw);
            cost += r * (S2 - S2 / (P / Pw));
        }
        return cost + halo;
    }
    uint32_t E = 0, ered = 0, ew = 0;
    for (uint32_t k = 0; k < dv.ndims; k++) {
        E += ex[k];
        if ((dv.reduce_mask >> k) & 1u) ered += ex[k];
        if ((dv.weight_mask >> k) & 1u) ew += ex[k];
    }
    uint64_t compute = (dv.flops + ((1ull << E) - 1)) >> E;
    uint32_t ek = E - ered;
    uint64_t part = (dv.keep_n + ((1ull << ek) - 1)) >> ek;
    uint64_t cost = compute + r * (((1ull << ered) - 1) * part);
    if (dv.weight_n) {
        const uint64_t S2 = 2 * ((dv.weight_n + ((1ull << ew) - 1)) >> ew);
        cost += r * (S2 - (S2 >> (E - ew)));
    }
    return cost + halo;
}

// Device byte of one configuration: the exponent sum log2(P) of power-of-two
// rows, else the device count P itself.
__device__ __forceinline__ uint32_t device_byte(const DevVertex &dv, const uint8_t *ex) {
    uint32_t x = dv.factors ? 1 : 0;
    for (uint32_t k = 0; k < dv.ndims; k++) x = dv.factors ? x * ex[k] : x + ex[k];
    return x;
}

// Split signature of one endpoint configuration of an edge: the split of every
// tensor dim (an unsplit dim counts as factor 1), one field per dim -- 5-bit
// exponents, or 8-bit factors.  Two endpoints redistribute nothing exactly when
// their signatures are equal.
__device__ __forceinline__ uint64_t split_signature(const int8_t *dims, uint32_t rank, const uint8_t *ex,
                                                   uint32_t factors) {
    const uint32_t w = factors ? 8 : 5, one = factors ? 1 : 0;
    uint64_t sig = 0;
    for (uint32_t k = 0; k < rank; k++) sig |= (uint64_t)(dims[k] >= 0 ? ex[dims[k]] : one) << (w * k);
    return sig;
}

// r * t_x of the volume-intersection model for one (producer config, consumer
// config) pair.  Device d of a configuration is the mixed-radix point of its
// split grid (loop dim 0 slowest); a tensor dim is cut into equal fractions on
// each side by the split of the loop dim it maps to (1 if unmapped).  Per
// tensor dim the parts of u and v are measured in units of 1/(s_u * s_v):
// v's part [x_v * s_u, (x_v + 1) * s_u), u's part [x_u * s_v, (x_u + 1) * s_v).
// forward  = max_d |need_v(d)| - |need_v(d) n hold_u(d)|, backward the same with
// u and v swapped; words = ceil(elems * fraction) per direction.  The host
// checks Q = prod s_u * s_v < 2^32, so every endpoint and volume in units fits
// 32 bits.  Devices that only one side uses contribute that side's whole part
// (a constant), so the walk covers the devices both use, as odometers over
// the two grids, and stops once both maxima reach their ceilings.
__device__ __forceinline__ uint64_t ceil_frac(uint64_t elems, uint64_t f, uint64_t Q) {
    // elems * f / Q rounded up, f <= Q < 2^32: (elems % Q) * f < Q^2 < 2^64
    const uint64_t q = elems / Q, rem = elems % Q;
    return q * f + (rem * f + Q - 1) / Q;
}

__device__ __forceinline__ uint32_t split_of(const DevVertex &x, const uint8_t *ex, int k) {
    return x.factors ? ex[k] : 1u << ex[k];
}

// With m = min over the devices both ends use of |need_v(d) n hold_u(d)|:
// forward = need_v - m (need_v when v uses more devices), backward = hold_u - m
// (hold_u when u uses more).  Per tensor dim the device's coordinate on each
// side advances every `stride` devices (the product of the splits of the loop
// dims after the mapped one) and wraps at the split; all per-dim state is
// indexed by unrolled constants so it stays in registers.
//
// Power-of-two splits take the closed form of k_edge_volume_pow2 instead.
__device__ __forceinline__ uint64_t volume_cost(const DevVertex &u, const uint8_t *exu, const DevVertex &v,
                                                const uint8_t *exv, const DevEdge &de, uint64_t r) {
    uint32_t Pu = 1, Pv = 1;
    for (uint32_t k = 0; k < u.ndims; k++) Pu *= split_of(u, exu, (int)k);
    for (uint32_t k = 0; k < v.ndims; k++) Pv *= split_of(v, exv, (int)k);
    uint32_t ta[kMaxDims], tb[kMaxDims], stu[kMaxDims], stv[kMaxDims];
    uint32_t xu[kMaxDims], xv[kMaxDims], pu[kMaxDims], pv[kMaxDims];
    uint32_t Q = 1, need_v = 1, hold_u = 1;
#pragma unroll
    for (int t = 0; t < kMaxDims; t++) {
        ta[t] = tb[t] = stu[t] = stv[t] = 1;
        xu[t] = xv[t] = pu[t] = pv[t] = 0;
        if (t < (int)de.rank) {
            const int ka = de.sdim[t], kb = de.ddim[t];
            if (ka >= 0) {
                ta[t] = split_of(u, exu, ka);
                for (int k = ka + 1; k < (int)u.ndims; k++) stu[t] *= split_of(u, exu, k);
            }
            if (kb >= 0) {
                tb[t] = split_of(v, exv, kb);
                for (int k = kb + 1; k < (int)v.ndims; k++) stv[t] *= split_of(v, exv, k);
            }
            Q *= ta[t] * tb[t];
            need_v *= ta[t];      // |v's part| = 1/b = a units
            hold_u *= tb[t];
        }
    }
    const uint32_t both = Pu < Pv ? Pu : Pv;
    uint32_t m = need_v < hold_u ? need_v : hold_u;
    for (uint32_t d = 0; d < both && m; d++) {
        uint32_t common = 1;
#pragma unroll
        for (int t = 0; t < kMaxDims; t++) {
            if (t < (int)de.rank) {
                const uint32_t a = ta[t], b = tb[t], cu = xu[t], cv = xv[t];
                const uint32_t lo = cv * a > cu * b ? cv * a : cu * b;
                const uint32_t hi = (cv + 1) * a < (cu + 1) * b ? (cv + 1) * a : (cu + 1) * b;
                common *= hi > lo ? hi - lo : 0;
                // next device
                if (++pu[t] == stu[t]) { pu[t] = 0; if (++xu[t] == ta[t]) xu[t] = 0; }
                if (++pv[t] == stv[t]) { pv[t] = 0; if (++xv[t] == tb[t]) xv[t] = 0; }
            }
        }
        m = common < m ? common : m;
    }
    const uint32_t fwd = Pv > Pu ? need_v : need_v - m, bwd = Pu > Pv ? hold_u : hold_u - m;
    return r * (ceil_frac(de.elems, fwd, Q) + ceil_frac(de.elems, bwd, Q));
}

// r * t_x from the two signatures and device bytes of the endpoints.
__device__ __forceinline__ uint64_t edge_cost_sig(uint64_t sig_a, uint64_t sig_b, uint32_t la, uint32_t lb,
                                                  uint64_t elems, uint64_t r, uint32_t factors) {
    if (sig_a == sig_b) return 0;
    uint32_t s = la > lb ? la : lb;
    if (factors) return r * ceil_div_u64(elems, s);
    return r * ((elems + ((1ull << s) - 1)) >> s);
}

// ------------------------------------------------------------------ prep: key-space blocks
// Batched launches: the workgroups of one launch are the concatenation of the
// workgroups of its vertices; find the vertex of this workgroup (uniform).
__device__ __forceinline__ uint32_t batch_find(const BatchEntry *__restrict__ be, uint32_t nbe, uint32_t wg) {
    uint32_t lo = 0, hi = nbe;
    while (hi - lo > 1) {
        uint32_t mid = (lo + hi) >> 1;
        if (be[mid].first <= wg) lo = mid; else hi = mid;
    }
    return __builtin_amdgcn_readfirstlane(lo);
}

// The small vertices of the bulk lane schedule (the chains of dependent
// vertices) run their waves at the highest issue priority: on a SIMD shared
// with the long fills of the bulk stream they then issue first.
__device__ __forceinline__ void set_priority(const BatchEntry &e) {
    if (e.prio) __builtin_amdgcn_s_setprio(3);
}

// The key of configuration c of vertex `me` under plan digits dv, summed over
// contributions [c0, c1): plain costs (layer, transfer) are summed in `sum`
// and shifted into key space at the end; DP tables are stored in this
// vertex's key space already; the layer term carries c into the low bits.
template <typename KeyT>
__device__ __forceinline__ typename KeyOps<KeyT>::Acc contrib_key(const Contrib *__restrict__ cb, uint32_t c0, uint32_t c1,
                                                const DevVertex &me, uint32_t c, const uint32_t (&dv)[kMaxDep],
                                                uint32_t bits, const DevVertex *__restrict__ V,
                                                const DevEdge *__restrict__ E, const uint64_t *__restrict__ L,
                                                const uint8_t *__restrict__ lsum, const uint64_t *__restrict__ sig,
                                                uint64_t r) {
    using Val = typename KeyOps<KeyT>::Val;
    using Acc = typename KeyOps<KeyT>::Acc;
    uint64_t sum = 0, low = 0;
    Acc keysum = 0;
    for (uint32_t k = c0; k < c1; k++) {
        const Contrib ct = cb[k];
        if (ct.kind == kContribLayer) {
            sum += L[me.L_off + c];
            low = c;
        } else if (ct.kind == kContribEdge) {
            const DevEdge de = E[ct.edge];
            const uint32_t xo = dv[ct.dig];
            const DevVertex ov = V[ct.vi_is_src ? de.dst : de.src];
            const uint64_t sme = sig[de.sig_off + (ct.vi_is_src ? 0 : V[de.src].K) + c];
            const uint64_t sot = sig[de.sig_off + (ct.vi_is_src ? me.K : 0) + xo];
            sum += edge_cost_sig(sme, sot, lsum[me.L_off + c], lsum[ov.L_off + xo], de.elems, r, de.factors);
        } else {
            uint64_t idx = (uint64_t)c * ct.sc;
            for (int k2 = 0; k2 < kMaxDep; k2++) idx += (uint64_t)dv[k2] * ct.sd[k2];
            if (ct.raw_u64) sum += ((const uint64_t *)ct.ptr)[idx];
            else keysum += KeyOps<KeyT>::val_to_acc(((const Val *)ct.ptr)[idx]);
        }
    }
    return ((Acc)sum << bits) + keysum + low;
}

// One workgroup handles `span` runs of kPrepThreads consecutive (c, column)
// elements of one outer index of one block, so the block, its contributions
// and the outer digits are uniform across the workgroup (scalar loads, which
// later runs find in the scalar cache); lanes differ only in (c, column).
template <typename KeyT>
__device__ __forceinline__ void prep_item(const PrepArgs &a, uint32_t wg, const DevVertex *__restrict__ V,
                                          const DevEdge *__restrict__ E, const uint64_t *__restrict__ L,
                                          const uint8_t *__restrict__ lsum, const uint64_t *__restrict__ sig,
                                          const Contrib *__restrict__ cb, uint64_t r) {
    KeyT *__restrict__ blocks = (KeyT *)a.blocks;
    uint32_t b = 0;
    while (b + 1 < a.nblocks && wg >= a.blk[b + 1].wg_begin) b++;
    b = __builtin_amdgcn_readfirstlane(b);
    const Block &bk = a.blk[b];
    const uint32_t rel = wg - bk.wg_begin;
    const uint32_t row = rel / bk.chunks, chunk = rel % bk.chunks;
    const uint32_t per_row = a.K * bk.ld;
    uint32_t dv[kMaxDep];
    for (int k = 0; k < kMaxDep; k++) dv[k] = 0;
    uint32_t x = row;
    for (int k = (int)bk.npre - 1; k >= 0; k--) {
        dv[bk.pre[k]] = x % bk.prerad[k];
        x /= bk.prerad[k];
    }
    const DevVertex me = V[a.vi];
    for (uint32_t s = 0; s < bk.span; s++) {
        const uint32_t e = (chunk * bk.span + s) * kPrepThreads + threadIdx.x;
        if (e >= per_row) return;
        const uint32_t c = e / bk.ld, q = e % bk.ld;
        KeyT *out = blocks + bk.out_off + (uint64_t)row * per_row + e;
        if (bk.post >= 0 && q >= bk.postrad) {
            *out = (KeyT)0;
            continue;
        }
        if (bk.post >= 0) dv[bk.post] = q;
        *out = KeyOps<KeyT>::from_acc(contrib_key<KeyT>(cb, bk.c_begin, bk.c_end, me, c, dv, a.bits, V, E, L,
                                                         lsum, sig, r));
    }
}

// Waits for every outstanding scalar-memory and LDS read (s_waitcnt
// lgkmcnt(0), other counters left alone).  Scalar loads return out of order,
// so a wait for one of them is always a wait for all of them: the pipelined
// loops wait for the operands of c *before* they request those of c + 1,
// otherwise the wait the compiler places before the first use of c's
// operands would also wait for the prefetch.
__device__ __forceinline__ void wait_lgkm_all() { __builtin_amdgcn_s_waitcnt(0xC07F); }

// ------------------------------------------------------------------ fill: row kernel
// Output T_i is laid out [z][o][r]: column digit z slowest, then the outer
// digits o (those sharing a lookup with z), then the row digits r.  A tile is
// TM x 64 consecutive rows of one (o, column chunk, c range); lane l holds
// rows l, l + 64, ...  For each c every row forms its operand a = sum of its
// row terms, and the wave reads the TZ column operands B[o][c][z0..z0+TZ)
// through the scalar unit (they are wave-uniform), so each cell is one add
// (SGPR operand) and one min; one scalar round trip per c feeds TM x 64 x TZ
// cells.  The four waves of a workgroup take the same tile and a quarter of
// its c range each, and combine their minima through LDS at the end: a wave
// then does a quarter of a tile's work, so a launch has four times as many,
// shorter, work items and its last partial round of waves costs little.
constexpr int kMergeVals = 16;   // values per lane moved through LDS per merge pass

template <typename KeyT>
using MergeBuf = KeyT[2][kMergeVals][64];

// Workgroup b of one vertex's row fill; xch: the workgroup's LDS merge buffer.
template <typename KeyT, int TZ, int TM, int NA>
__device__ __forceinline__ void rows_item(const RowsArgs &a, uint32_t b, MergeBuf<KeyT> &xch) {
    using Ops = KeyOps<KeyT>;
    using Val = typename Ops::Val;
    const uint32_t lane = threadIdx.x & 63;
    // the wave index is uniform across the wave: say so, so that everything
    // derived from it (c range, column addresses) lives in SGPRs
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // blocks are dealt round-robin to the 8 XCDs: give every XCD a contiguous
    // range of tiles so that tiles sharing a column slice share an L2 (every
    // vertex's block count and first block are multiples of 8, so the XCD of
    // a block is its local index mod 8)
    const uint32_t nb = a.nblocks_launched;
    const uint64_t wg = (uint64_t)(b % 8) * (nb / 8) + b / 8;
    // a workgroup takes 4 / P tiles, P = a.parts waves per tile, each wave a
    // P-th of the tile's c range
    const uint32_t P = a.parts, tpw = 4 / P;
    if (wg * tpw >= a.total_tiles) return;   // the whole workgroup leaves together
    const uint32_t part = wave % P, tin = wave / P;
    const bool has_tile = wg * tpw + tin < a.total_tiles;
    // (a wave without a tile computes nothing but still takes part in the merge)
    const uint64_t tile = min(wg * tpw + tin, a.total_tiles - 1);
    // tile order (fastest first): row tile, column chunk, outer index, c split --
    // all chunks of one outer index run close together and share its slices
    const uint32_t rowtile = (uint32_t)(tile % a.tiles_per_o);
    uint64_t t2 = tile / a.tiles_per_o;
    const uint32_t chunk = (uint32_t)(t2 % a.nchunks);
    t2 /= a.nchunks;
    const uint32_t o = (uint32_t)(t2 % a.MO);
    const uint32_t split = (uint32_t)(t2 / a.MO);

    constexpr int NT = NA < 0 ? kMaxATerms : NA;
    constexpr int NTA = NT > 0 ? NT : 1;
    const int na = NA < 0 ? (int)a.na : NA;
    uint32_t dO[kMaxDep];
    {
        uint32_t x = o;
        for (int k = kMaxDep - 1; k >= 0; k--)
            if (k < (int)a.nO) { dO[k] = x % a.radO[k]; x /= a.radO[k]; } else dO[k] = 0;
    }
    // row terms are read with buffer loads: per-lane byte offset in a VGPR,
    // the c-dependent part as a scalar offset, no per-c address arithmetic
    __amdgpu_buffer_rsrc_t rsrc[NTA];
    uint32_t tsc[NTA];
#pragma unroll
    for (int t = 0; t < NTA; t++) {
        rsrc[t] = __builtin_amdgcn_make_buffer_rsrc(t < na ? const_cast<void *>(a.a[t].ptr) : nullptr, (short)0,
                                                    t < na ? (int)a.a[t].bytes : 0, kBufferWord3);
        tsc[t] = t < na ? a.a[t].sc * (uint32_t)sizeof(Val) : 0;
    }
    uint32_t r[TM], offb[TM][NTA];
    bool valid[TM];
#pragma unroll
    for (int m = 0; m < TM; m++) {
        r[m] = (rowtile * TM + m) * 64 + lane;
        valid[m] = r[m] < a.MR;
        uint32_t x = valid[m] ? r[m] : a.MR - 1, dR[kMaxDep];
        for (int k = kMaxDep - 1; k >= 0; k--)
            if (k < (int)a.nR) { dR[k] = x % a.radR[k]; x /= a.radR[k]; } else dR[k] = 0;
#pragma unroll
        for (int t = 0; t < NTA; t++) {
            uint32_t off = 0;
            if (t < na)
                for (int k = 0; k < kMaxDep; k++) off += dO[k] * a.a[t].sdO[k] + dR[k] * a.a[t].sdR[k];
            offb[m][t] = off * (uint32_t)sizeof(Val);
        }
    }
    // this wave's part [c0, c1) of the tile's c range (possibly empty)
    const uint32_t cs = split * a.cper, ce_ = has_tile ? min(a.K, cs + a.cper) : cs;
    const uint32_t q = (ce_ - cs + P - 1) / P;
    const uint32_t c0 = min(ce_, cs + part * q), c1 = min(ce_, c0 + q);
    const uint32_t ldz = a.ldz;
    const KeyT *B = (const KeyT *)a.B + (uint64_t)o * a.K * ldz + (uint64_t)chunk * TZ;

    KeyT acc[TM][TZ];
#pragma unroll
    for (int m = 0; m < TM; m++)
#pragma unroll
        for (int t = 0; t < TZ; t++) acc[m][t] = Ops::sentinel();

    // Software pipeline over two register sets of U values of c each: the
    // row terms and column chunks of the next U values are requested while
    // the cells of the current ones are computed from the other set, so load
    // latency overlaps VALU work.  Narrow tiles have little work per c and
    // keep U = 4 values in flight per set; 8-column tiles keep 2 (two sets of
    // 2 x 8 keys still fit in SGPRs) -- they serve the small, latency-bound
    // vertices, whose waves otherwise wait out a round trip per c.  Loads past
    // c1 repeat column c1 - 1 (in bounds, unused) so that every load is
    // unconditional and the register sets never need copying.
    constexpr int U = TZ <= 2 ? 4 : TZ <= 8 ? 2 : 1;
    using SKey = const __attribute__((address_space(4))) KeyT;
    uint64_t xe[U][TM][NTA], xo[U][TM][NTA];
    KeyT ce[U][TZ], co[U][TZ];
    auto load = [&](uint64_t (&xs)[U][TM][NTA], KeyT (&bs)[U][TZ], uint32_t cc) {
#pragma unroll
        for (int u = 0; u < U; u++) {
            const uint32_t cu = min(cc + u, c1 - 1);
#pragma unroll
            for (int m = 0; m < TM; m++)
#pragma unroll
                for (int t = 0; t < NTA; t++)
                    if (t < na)
                        xs[u][m][t] = __builtin_bit_cast(uint64_t, __builtin_amdgcn_raw_buffer_load_b64(
                                                                       rsrc[t], (int)offb[m][t], (int)(cu * tsc[t]), 0));
            SKey *brow = (SKey *)(uintptr_t)(B + (uint64_t)cu * ldz);
#pragma unroll
            for (int t = 0; t < TZ; t++) bs[u][t] = brow[t];
        }
    };
    auto cells = [&](const uint64_t (&xs)[U][TM][NTA], const KeyT (&bs)[U][TZ], uint32_t n) {
#pragma unroll
        for (int u = 0; u < U; u++) {
            if (u > 0 && (uint32_t)u >= n) break;
            KeyT av[TM];
#pragma unroll
            for (int m = 0; m < TM; m++) {
                av[m] = (KeyT)0;
#pragma unroll
                for (int t = 0; t < NTA; t++)
                    if (t < na) {
                        const KeyT v = __builtin_bit_cast(KeyT, xs[u][m][t]);
                        av[m] = t == 0 ? v : Ops::add(av[m], v);
                    }
            }
#pragma unroll
            for (int t = 0; t < TZ; t++)
#pragma unroll
                for (int m = 0; m < TM; m++) acc[m][t] = Ops::min(acc[m][t], Ops::add(av[m], bs[u][t]));
        }
    };
    if (c0 < c1) {
        load(xe, ce, c0);
        uint32_t c = c0;
        for (; c + U < c1; c += 2 * U) {
            // up to 16 columns both sets fit in SGPRs at once: the barriers
            // keep the scheduler from sinking the loads of the next set below
            // the cells of the current one, and the explicit wait for the
            // current operands comes before those loads are issued
            if constexpr (TZ <= 16) {
                wait_lgkm_all();
                __builtin_amdgcn_sched_barrier(0);
            }
            load(xo, co, c + U);
            if constexpr (TZ <= 16) __builtin_amdgcn_sched_barrier(0);
            cells(xe, ce, U);
            if constexpr (TZ <= 16) {
                wait_lgkm_all();
                __builtin_amdgcn_sched_barrier(0);
            }
            load(xe, ce, c + 2 * U);
            if constexpr (TZ <= 16) __builtin_amdgcn_sched_barrier(0);
            cells(xo, co, min((uint32_t)U, c1 - (c + U)));
        }
        if (c < c1) cells(xe, ce, min((uint32_t)U, c1 - c));
    }

    // combine the parts of a tile through LDS, halving the number of holders
    // per stage (P = 4: parts 2, 3 -> 0, 1, then 1 -> 0; P = 2: 1 -> 0),
    // kMergeVals values per lane and pass; P is uniform across the workgroup,
    // so every wave meets the same barriers
    constexpr int V = TM * TZ;
    for (uint32_t d = P / 2; d >= 1; d /= 2) {
#pragma unroll
        for (int p0 = 0; p0 < V; p0 += kMergeVals) {
            constexpr int W = kMergeVals;
            __syncthreads();
            if (part >= d && part < 2 * d) {
                const uint32_t slot = tin * d + (part - d);
#pragma unroll
                for (int j = 0; j < W; j++)
                    if (p0 + j < V) xch[slot][j][lane] = acc[(p0 + j) / TZ][(p0 + j) % TZ];
            }
            __syncthreads();
            if (part < d) {
                const uint32_t slot = tin * d + part;
#pragma unroll
                for (int j = 0; j < W; j++)
                    if (p0 + j < V) {
                        KeyT &x = acc[(p0 + j) / TZ][(p0 + j) % TZ];
                        x = Ops::min(x, xch[slot][j][lane]);
                    }
            }
        }
    }
    if (part != 0 || !has_tile) return;

    const uint64_t plane = (uint64_t)a.MO * a.MR;
    const uint32_t zbase = chunk * TZ;
    // fused minimum of the reader v_j (c_j = z): per row, its keys over this
    // tile's columns -- the stored value of T[z][r] (already in v_j's key
    // space) plus v_j's other row terms at (r, z) and its column block at z
    // -- reduced in the lane, then min-combined across tiles atomically
    constexpr bool kFuse = sizeof(KeyT) == 8;
    const bool fuse = kFuse && a.fz_keys != nullptr;
#pragma unroll
    for (int m = 0; m < TM; m++) {
        if (!valid[m]) continue;
        const uint64_t base_idx = (uint64_t)o * a.MR + r[m];
        uint32_t fzoff[kMaxATerms];
        KeyT best = Ops::sentinel();
        if (fuse) {
            uint32_t x = r[m], dR[kMaxDep];
            for (int k = kMaxDep - 1; k >= 0; k--)
                if (k < (int)a.nR) { dR[k] = x % a.radR[k]; x /= a.radR[k]; } else dR[k] = 0;
            for (int q = 0; q < kMaxATerms; q++) {
                uint32_t off = 0;
                if (q < (int)a.fz_na)
                    for (int k = 0; k < kMaxDep; k++) off += dR[k] * a.fz_a[q].sdR[k];
                fzoff[q] = off;
            }
        }
#pragma unroll
        for (int t = 0; t < TZ; t++) {
            const uint32_t z = zbase + t;
            if (z < a.Kz) {
                const uint64_t idx = (uint64_t)z * plane + base_idx;
                if (a.nsplit > 1) {
                    ((KeyT *)a.partial)[(uint64_t)split * a.N + idx] = acc[m][t];
                } else {
                    Val v;
                    uint32_t cc;
                    Ops::split(acc[m][t], a.bits, a.out_shift, v, cc);
                    if (a.T) ((Val *)a.T)[idx] = v;
                    a.A[idx] = (uint16_t)cc;
                    if constexpr (kFuse) {
                        if (fuse) {
                            KeyT k = __builtin_bit_cast(KeyT, v);
                            for (int q = 0; q < kMaxATerms; q++)
                                if (q < (int)a.fz_na)
                                    k = Ops::add(k, ((const KeyT *)a.fz_a[q].ptr)[fzoff[q] + z * a.fz_a[q].sc]);
                            k = Ops::add(k, ((const KeyT *)a.fz_B)[(uint64_t)z * a.fz_ldz]);
                            best = Ops::min(best, k);
                        }
                    }
                }
            }
        }
        if constexpr (kFuse) {
            if (fuse)
                atomicMin((unsigned long long *)a.fz_keys + r[m],
                          (unsigned long long)__builtin_bit_cast(uint64_t, best));
        }
    }
}

template <typename KeyT>
__device__ __forceinline__ void reduce_item(const ReduceArgs &a, uint32_t lb) {
    using Ops = KeyOps<KeyT>;
    using Val = typename Ops::Val;
    for (uint64_t t = lb * (uint64_t)blockDim.x + threadIdx.x; t < a.N; t += (uint64_t)a.nblk * blockDim.x) {
        KeyT best = ((const KeyT *)a.partial)[t];
        for (uint32_t s = 1; s < a.nsplit; s++) best = Ops::min(best, ((const KeyT *)a.partial)[s * a.N + t]);
        Val v;
        uint32_t cc;
        Ops::split(best, a.bits, a.out_shift, v, cc);
        ((Val *)a.T)[t] = v;
        a.A[t] = (uint16_t)cc;
    }
}

// ------------------------------------------------------------------ fill: generic kernel
// Any |D(i)| <= PASE_MAX_DEP and any term shapes.  A group of 2^group_log2
// lanes owns one entry phi: lane l evaluates c = l, l + G, ... (key = sum of
// the terms), the group then takes the minimum key with cross-lane swaps.
// Keys are distinct for distinct c, so the minimum -- and with it the lowest
// optimal c -- does not depend on the evaluation order.
template <typename KeyT>
__device__ __forceinline__ KeyT shfl_xor_key(KeyT v, int mask) {
    constexpr int W = sizeof(KeyT) / 4;   // 32-bit words of a key
    struct Words { uint32_t w[W]; };
    Words x = __builtin_bit_cast(Words, v);
#pragma unroll
    for (int k = 0; k < W; k++) x.w[k] = (uint32_t)__shfl_xor((int)x.w[k], mask, 64);
    return __builtin_bit_cast(KeyT, x);
}

template <typename KeyT, int NT>
__device__ __forceinline__ void generic_item(const GenericArgs &a, uint32_t lb) {
    using Ops = KeyOps<KeyT>;
    using Val = typename Ops::Val;
    const uint32_t G = 1u << a.group_log2;
    const uint64_t nthreads = (uint64_t)a.N << a.group_log2;
    constexpr int MT = NT < 0 ? kMaxGTerms : NT;
    const int nt = NT < 0 ? (int)a.nt : NT;
    for (uint64_t tid = lb * (uint64_t)blockDim.x + threadIdx.x; tid < ((nthreads + 255) / 256) * 256;
         tid += (uint64_t)a.nblk * blockDim.x) {
        const bool live = tid < nthreads;
        const uint64_t phi = live ? tid >> a.group_log2 : a.N - 1;
        const uint32_t lane = (uint32_t)(tid & (G - 1));
        uint32_t d[kMaxDep];
        uint64_t x = phi;
        for (int k = kMaxDep - 1; k >= 0; k--)
            if (k < (int)a.m) { d[k] = (uint32_t)(x % a.rad[k]); x /= a.rad[k]; } else d[k] = 0;
        const KeyT *base[MT];
        uint32_t sc[MT];
#pragma unroll
        for (int t = 0; t < MT; t++) {
            uint64_t o = 0;
            if (t < nt)
                for (int k = 0; k < kMaxDep; k++) o += (uint64_t)d[k] * a.t[t].sd[k];
            base[t] = (const KeyT *)a.t[t < nt ? t : 0].ptr + (t < nt ? o : 0);
            sc[t] = t < nt ? a.t[t].sc : 0;
        }
        KeyT best0 = Ops::sentinel(), best1 = Ops::sentinel();
        uint32_t c = lane;
        // two independent chains keep two loads of every term in flight
        for (; c + G < a.K; c += 2 * G) {
            KeyT k0 = base[0][(uint64_t)c * sc[0]];
            KeyT k1 = base[0][(uint64_t)(c + G) * sc[0]];
#pragma unroll
            for (int t = 1; t < MT; t++)
                if (t < nt) {
                    k0 = Ops::add(k0, base[t][(uint64_t)c * sc[t]]);
                    k1 = Ops::add(k1, base[t][(uint64_t)(c + G) * sc[t]]);
                }
            best0 = Ops::min(best0, k0);
            best1 = Ops::min(best1, k1);
        }
        if (c < a.K) {
            KeyT k0 = base[0][(uint64_t)c * sc[0]];
#pragma unroll
            for (int t = 1; t < MT; t++)
                if (t < nt) k0 = Ops::add(k0, base[t][(uint64_t)c * sc[t]]);
            best0 = Ops::min(best0, k0);
        }
        KeyT best = Ops::min(best0, best1);
        for (uint32_t m = G >> 1; m > 0; m >>= 1) best = Ops::min(best, shfl_xor_key(best, (int)m));
        if (live && lane == 0) {
            Val v;
            uint32_t cc;
            Ops::split(best, a.bits, a.out_shift, v, cc);
            ((Val *)a.T)[phi] = v;
            a.A[phi] = (uint16_t)cc;
        }
    }
}

// ------------------------------------------------------------------ direct fill (small vertices)
// Like the generic fill, 2^group_log2 lanes share one table entry and stride
// over c.  Each lane first resolves every contribution for its entry once --
// an array read at base + c * stride (layer costs, caller or volume edge
// matrices, producer tables) or a split-signature edge term with the other
// endpoint's signature and device byte fixed -- so the loop over c only loads
// data.  Vertices with more contributions than fit the register set take the
// per-cell path of the prep kernel.
constexpr int kDirectTerms = 8;

template <typename KeyT>
__device__ __forceinline__ void direct_item(const DirectArgs &a, uint32_t lb, const DevVertex *__restrict__ V,
                                            const DevEdge *__restrict__ E, const uint64_t *__restrict__ L,
                                            const uint8_t *__restrict__ lsum, const uint64_t *__restrict__ sig,
                                            const Contrib *__restrict__ cb, uint64_t r, KeyT (&xch)[4]) {
    using Ops = KeyOps<KeyT>;
    using Val = typename Ops::Val;
    const uint32_t G = 1u << a.group_log2;
    const uint64_t nthreads = (uint64_t)a.N << a.group_log2;
    const DevVertex me = V[a.vi];
    const uint32_t nt = a.c_end - a.c_begin;
    const bool fast = nt <= (uint32_t)kDirectTerms;
    for (uint64_t tid = lb * (uint64_t)blockDim.x + threadIdx.x; tid < ((nthreads + 255) / 256) * 256;
         tid += (uint64_t)a.nblk * blockDim.x) {
        const bool live = tid < nthreads;
        const uint64_t phi = live ? tid >> a.group_log2 : a.N - 1;
        const uint32_t lane = (uint32_t)(tid & (G - 1));
        uint32_t dv[kMaxDep];
        uint64_t x = phi;
        for (int k = kMaxDep - 1; k >= 0; k--)
            if (k < (int)a.m) { dv[k] = (uint32_t)(x % a.rad[k]); x /= a.rad[k]; } else dv[k] = 0;
        KeyT best = Ops::sentinel();
        if (fast) {
            // kind: 0 plain u64 array, 1 key-space table, 2 signature edge
            const char *base[kDirectTerms];
            uint32_t stride[kDirectTerms], kind[kDirectTerms], lot[kDirectTerms], fac[kDirectTerms];
            const uint8_t *lme[kDirectTerms];
            uint64_t sot[kDirectTerms], elems[kDirectTerms];
#pragma unroll
            for (int t = 0; t < kDirectTerms; t++) {
                base[t] = nullptr;
                lme[t] = nullptr;
                stride[t] = kind[t] = lot[t] = fac[t] = 0;
                sot[t] = elems[t] = 0;
                if (t < (int)nt) {
                    const Contrib ct = cb[a.c_begin + t];
                    if (ct.kind == kContribLayer) {
                        base[t] = (const char *)(L + me.L_off);
                        stride[t] = 8;
                    } else if (ct.kind == kContribEdge) {
                        const DevEdge de = E[ct.edge];
                        const uint32_t xo = dv[ct.dig];
                        const DevVertex ov = V[ct.vi_is_src ? de.dst : de.src];
                        kind[t] = 2;
                        base[t] = (const char *)(sig + de.sig_off + (ct.vi_is_src ? 0 : V[de.src].K));
                        stride[t] = 8;
                        sot[t] = sig[de.sig_off + (ct.vi_is_src ? me.K : 0) + xo];
                        lme[t] = lsum + me.L_off;
                        lot[t] = lsum[ov.L_off + xo];
                        elems[t] = de.elems;
                        fac[t] = de.factors;
                    } else {
                        uint64_t idx = 0;
                        for (int k2 = 0; k2 < kMaxDep; k2++) idx += (uint64_t)dv[k2] * ct.sd[k2];
                        kind[t] = ct.raw_u64 ? 0 : 1;
                        stride[t] = ct.sc * 8;
                        base[t] = (const char *)ct.ptr + idx * 8;
                    }
                }
            }
            for (uint32_t c = lane; c < a.K; c += G) {
                uint64_t sum = 0, keysum = 0;
#pragma unroll
                for (int t = 0; t < kDirectTerms; t++) {
                    if (t < (int)nt) {
                        if (kind[t] == 2) {
                            const uint64_t sme = *(const uint64_t *)(base[t] + (uint64_t)c * stride[t]);
                            sum += edge_cost_sig(sme, sot[t], lme[t][c], lot[t], elems[t], r, fac[t]);
                        } else {
                            const uint64_t v = *(const uint64_t *)(base[t] + (uint64_t)c * stride[t]);
                            if (kind[t] == 0) sum += v;
                            else keysum += Ops::val_to_u64(__builtin_bit_cast(Val, v));
                        }
                    }
                }
                // the layer term is always present: c fills the low bits
                best = Ops::min(best, Ops::from_u64((sum << a.bits) + keysum + c));
            }
        } else {
            for (uint32_t c = lane; c < a.K; c += G)
                best = Ops::min(best, Ops::from_acc(contrib_key<KeyT>(cb, a.c_begin, a.c_end, me, c, dv, a.bits, V,
                                                                      E, L, lsum, sig, r)));
        }
        for (uint32_t m = (G < 64 ? G : 64) >> 1; m > 0; m >>= 1) best = Ops::min(best, shfl_xor_key(best, (int)m));
        if (G > 64) {
            // a group of 2 or 4 waves: their minima meet in LDS (every thread
            // of the workgroup runs the same iterations, so the barriers match)
            const uint32_t wave = threadIdx.x >> 6;
            if ((threadIdx.x & 63) == 0) xch[wave] = best;
            __syncthreads();
            if (lane == 0)
                for (uint32_t w = 1; w < G / 64; w++) best = Ops::min(best, xch[wave + w]);
            __syncthreads();
        }
        if (live && lane == 0) {
            Val v;
            uint32_t cc;
            Ops::split(best, a.bits, a.out_shift, v, cc);
            ((Val *)a.T)[phi] = v;
            a.A[phi] = (uint16_t)cc;
        }
    }
}

// ------------------------------------------------------------------ class fill
// Pointers read from a descriptor are generic to the compiler, which then
// issues flat loads (they also count as LDS operations and wait for them);
// these name global memory.
template <typename T> using Glb = __attribute__((address_space(1))) T *;
template <typename T> __device__ __forceinline__ Glb<const T> glb(const void *p) { return (Glb<const T>)(uintptr_t)p; }

// Class table of one edge shape: every configuration's place in the order of
// (signature, index) and, per configuration of the other end, the range of
// u's configurations with its signature, by counting: kClassTabLanes threads
// per configuration, each against its share of all signatures (staged through
// LDS).  A share of 1/16 keeps the loop at 58 of the Transformer's 924
// signatures per edge (one thread per configuration took 53 us).
constexpr uint32_t kClassTabTile = 1024;
__device__ __forceinline__ void class_table_item(const DevClassTab &t, uint32_t lb, const uint8_t *__restrict__ ex,
                                                 char *__restrict__ ws, uint64_t (&buf)[kClassTabTile]) {
    const uint32_t n = t.K + t.Kz, sub = threadIdx.x % kClassTabLanes;
    const uint32_t e = lb * (256 / kClassTabLanes) + threadIdx.x / kClassTabLanes;
    auto sig_of = [&](uint32_t i) {
        return i < t.K ? split_signature(t.udim, t.rank, ex + t.ex_u + (uint64_t)i * t.ndu, t.factors)
                       : split_signature(t.zdim, t.rank, ex + t.ex_z + (uint64_t)(i - t.K) * t.ndz, t.factors);
    };
    const uint64_t me = e < n ? sig_of(e) : 0;
    uint32_t ulow = 0, ueq = 0, ueqb = 0, zlow = 0, zeqb = 0;   // smaller, equal, equal and before, per end
    for (uint32_t base = 0; base < n; base += kClassTabTile) {
        __syncthreads();
        for (uint32_t i = threadIdx.x; i < kClassTabTile && base + i < n; i += 256) buf[i] = sig_of(base + i);
        __syncthreads();
        for (uint32_t j = sub; j < kClassTabTile && base + j < n; j += kClassTabLanes) {
            const uint64_t s = buf[j];
            const bool lt = s < me, eq = s == me, before = eq && base + j < e, u = base + j < t.K;
            ulow += lt && u;
            ueq += eq && u;
            ueqb += before && u;
            zlow += lt && !u;
            zeqb += before && !u;
        }
    }
    for (uint32_t m = kClassTabLanes / 2; m > 0; m >>= 1) {
        ulow += __shfl_xor(ulow, m, 64);
        ueq += __shfl_xor(ueq, m, 64);
        ueqb += __shfl_xor(ueqb, m, 64);
        zlow += __shfl_xor(zlow, m, 64);
        zeqb += __shfl_xor(zeqb, m, 64);
    }
    if (sub) return;
    if (e < t.K) {
        ((uint16_t *)(ws + t.inv_off))[e] = (uint16_t)(ulow + ueqb);
        ((uint16_t *)(ws + t.perm_off))[ulow + ueqb] = (uint16_t)e;
        ((uint16_t *)(ws + t.first_off))[e] = (uint16_t)ulow;
    } else if (e < n) {
        ((ClassEntry *)(ws + t.zs_off))[zlow + zeqb] = ClassEntry{(uint16_t)ulow, (uint16_t)ueq, e - t.K};
        ((uint32_t *)(ws + t.zr_off))[e - t.K] = ulow | ueq << 16;
    }
}

// Workgroup lb of one vertex's class fill: 2^lr rows (the fastest bits of the
// thread index) x blockDim >> lr groups of lanes.
//
// Few rows (class_item_small): every configuration's data is read by one group
// only, so each thread loads it where it needs it; LDS holds X alone (a few
// KB, so the workgroup fits beside those of a large fill on another stream).
// All loads of a thread are independent (U configurations and entries in
// flight): about three memory round trips in all.
// A lookup's value as a key; raw: a plain integer cost read through the table's
// type (keys of 64 bits only, the same width).
template <typename KeyT>
__device__ __forceinline__ KeyT class_term(uint32_t raw, uint32_t bits, typename KeyOps<KeyT>::Val v) {
    if (raw) return KeyOps<KeyT>::from_u64(__builtin_bit_cast(uint64_t, v) << bits);
    return __builtin_bit_cast(KeyT, v);
}

template <typename KeyT, int NE, int NT>
__device__ __forceinline__ void class_item_small(const ClassArgs &a, uint32_t lb, char *lds) {
    using Ops = KeyOps<KeyT>;
    using Val = typename Ops::Val;
    constexpr int ME = NE > 0 ? NE : 1, MT = NT > 0 ? NT : 1;
    constexpr int U = NE + NT <= 2 ? 4 : 2;   // configurations in flight per thread (registers)
    const uint32_t threads = blockDim.x, lr = a.lr, R = 1u << lr, G = threads >> lr, K = a.K, Kz = a.Kz;
    const bool has_z = a.has_z;
    const uint32_t rl = threadIdx.x & (R - 1), g = threadIdx.x >> lr;
    const uint32_t row = lb * R + rl, rows = a.rows, bits = a.bits, out_shift = a.out_shift;
    const bool live = row < rows;
    KeyT *red = (KeyT *)lds;                            // [waves][R][2]
    KeyT *X = red + (threads / 64) * R * 2;             // [K][R]
    const Glb<Val> T = (Glb<Val>)(uintptr_t)a.T;
    const Glb<uint16_t> A = (Glb<uint16_t>)(uintptr_t)a.A;
    const Glb<const KeyT> Lk = glb<KeyT>(a.Lk), fzc = glb<KeyT>(a.fzc), fzo = glb<KeyT>(a.fzo);
    const Glb<const uint16_t> inv = glb<uint16_t>(a.inv);
    const Glb<const uint64_t> zs = glb<uint64_t>(a.zs);   // ClassEntry: first, count, z

    uint32_t d[kMaxDep];
    {
        uint32_t x = live ? row : rows - 1;
        for (int k = kMaxDep - 1; k >= 0; k--)
            if (k < (int)a.nR) {
                d[k] = k ? x % a.rad[k] : x;
                if (k) x /= a.rad[k];
            } else d[k] = 0;
    }
    uint64_t so[ME];
    KeyT fo[ME];
    Glb<const uint64_t> sc[ME];
    Glb<const KeyT> fc[ME];
    Glb<const Val> tp[MT];
    uint32_t tsc[MT];
#pragma unroll
    for (int t = 0; t < NE; t++) {
        uint32_t w = 0;
        for (int k = 0; k < kMaxDep; k++) w = k == (int)a.e[t].dig ? d[k] : w;
        so[t] = glb<uint64_t>(a.e[t].sig_o)[w];
        fo[t] = glb<KeyT>(a.e[t].f_o)[w];
        sc[t] = glb<uint64_t>(a.e[t].sig_c);
        fc[t] = glb<KeyT>(a.e[t].f_c);
    }
#pragma unroll
    for (int t = 0; t < NT; t++) {
        uint32_t o = 0;
        for (int k = 0; k < kMaxDep; k++)
            if (k < (int)a.nR) o += d[k] * a.t[t].sd[k];
        tp[t] = glb<Val>(a.t[t].ptr) + o;
        tsc[t] = a.t[t].sc;
    }
    // the first entries of z of this group, requested ahead of the barrier
    uint64_t w[U];
    KeyT fz[U];
    if (has_z) {
#pragma unroll
        for (int u = 0; u < U; u++) w[u] = zs[min(g + u * G, Kz - 1)];
    }
    KeyT m0 = Ops::sentinel(), m1 = Ops::sentinel();
    for (uint32_t c0 = g; c0 < K; c0 += U * G) {
        KeyT x[U], f[U], ef[U][ME], tv[U][MT];
        uint64_t es[U][ME];
        uint32_t at[U];
#pragma unroll
        for (int u = 0; u < U; u++) {
            // (past the end: the last configuration once more, the same minima and store)
            const uint32_t c = min(c0 + u * G, K - 1);
            x[u] = Lk[c];
            if (has_z) {
                at[u] = inv[c];
                f[u] = fzc[c];
            }
#pragma unroll
            for (int t = 0; t < NE; t++) {
                es[u][t] = sc[t][c];
                ef[u][t] = fc[t][c];
            }
#pragma unroll
            for (int t = 0; t < NT; t++) tv[u][t] = class_term<KeyT>(a.t[t].raw, bits, tp[t][(uint64_t)c * tsc[t]]);
        }
#pragma unroll
        for (int u = 0; u < U; u++) {
#pragma unroll
            for (int t = 0; t < NE; t++)
                x[u] = Ops::add(x[u], es[u][t] == so[t] ? (KeyT)0 : Ops::min(ef[u][t], fo[t]));
#pragma unroll
            for (int t = 0; t < NT; t++) x[u] = Ops::add(x[u], tv[u][t]);
            m0 = Ops::min(m0, x[u]);
            if (has_z) {
                m1 = Ops::min(m1, Ops::add(x[u], f[u]));
                X[(at[u] << lr) + rl] = x[u];
            }
        }
    }
    if (has_z) {
#pragma unroll
        for (int u = 0; u < U; u++) fz[u] = fzo[w[u] >> 32];
    }
    for (uint32_t m = R; m < 64; m <<= 1) {
        m0 = Ops::min(m0, shfl_xor_key(m0, (int)m));
        m1 = Ops::min(m1, shfl_xor_key(m1, (int)m));
    }
    const uint32_t RW = min(R, 64u), wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if (lane < RW) {
        red[(wave * RW + lane) * 2] = m0;
        red[(wave * RW + lane) * 2 + 1] = m1;
    }
    __syncthreads();
    for (uint32_t v = 0; v < threads / 64; v++) {
        m0 = Ops::min(m0, red[(v * RW + rl) * 2]);
        m1 = Ops::min(m1, red[(v * RW + rl) * 2 + 1]);
    }
    if (!live) return;
    auto put = [&](uint64_t idx, KeyT key) {
        Val v;
        uint32_t cc;
        Ops::split(key, bits, out_shift, v, cc);
        T[idx] = v;
        A[idx] = (uint16_t)cc;
    };
    if (!has_z) {
        if (g == 0) put(row, m0);
        return;
    }
    for (uint32_t q0 = g; q0 < Kz; q0 += U * G) {
        if (q0 != g) {
#pragma unroll
            for (int u = 0; u < U; u++) w[u] = zs[min(q0 + u * G, Kz - 1)];
#pragma unroll
            for (int u = 0; u < U; u++) fz[u] = fzo[w[u] >> 32];
        }
#pragma unroll
        for (int u = 0; u < U; u++) {
            if (q0 + u * G >= Kz) break;
            const uint32_t first = (uint32_t)w[u] & 0xffff, count = (uint32_t)w[u] >> 16;
            KeyT best = Ops::min(m1, Ops::add(m0, fz[u]));
            for (uint32_t k = 0; k < count; k++) best = Ops::min(best, X[((first + k) << lr) + rl]);
            put((w[u] >> 32) * rows + row, best);
        }
    }
}

// Many rows (class_item_staged): first the workgroup brings the per-configuration data (layer cost, f, the
// rest edges' signatures and f) into LDS in class order, and the class entries
// of z: both are read many times, by all rows, and the class order makes every
// later index a sequential one.  Then the groups share the configurations c:
// X[c][row] is formed for its two minima, min X and min (X + f(c)), and kept
// in LDS when `keep`.  After these are combined (lane swaps, LDS) the groups
// share the configurations z in class order: a table entry is the minimum of
// its class's X values and of the two minima.  When X of all K configurations
// does not fit (keep = 0; 64 rows, one wave per group) each class's X values are
// formed again: one more evaluation per (c, row), against Kz / K table entries.
//
// Bound by the stores of its table (10 bytes per entry) where its lookups are
// small: 1.8e7 entries of the Transformer at p = 64 in 47 us, 3.8 TB/s, with
// the VALU busy for 31% of its cycles; 1.1e8 at p = 24 in 278 us, 4.0 TB/s.
// With a lookup of the table's size its loads are waited for as well: 78 us
// (2.3 TB/s, waves waiting for 69% of their cycles) and 569 us.
//
// Against the dense fill: four leaves of 8.3e9 cells and 32 small ones 2.05 ms
// dense (94% of the fp64 issue rate) and 0.24 ms here, before the four were
// taken into joint fills; one level of the encoder chain 20 us (prep, row fill,
// split reduction) and 6 us.  With the data read from global memory by every
// group instead of staged, those leaves took 0.57 ms (vector loads of data that
// whole waves share).
template <typename KeyT, int NE, int NT>
__device__ __forceinline__ void class_item_staged(const ClassArgs &a, uint32_t lb, char *lds) {
    using Ops = KeyOps<KeyT>;
    using Val = typename Ops::Val;
    constexpr int ME = NE > 0 ? NE : 1, MT = NT > 0 ? NT : 1;
    constexpr int U = NE + NT <= 2 ? 4 : 2;   // configurations in flight per thread (registers)
    struct alignas(16) Rec { KeyT x, f; };              // layer cost and f of a configuration (edge: signature and f)
    struct alignas(16) EdgeRec { uint64_t sig; KeyT f; };
    struct alignas(16) ZRec { uint32_t place, z; KeyT f; };   // place: first | count << 16
    const uint32_t threads = blockDim.x, lr = a.lr, R = 1u << lr, G = threads >> lr, K = a.K, Kz = a.Kz;
    const bool has_z = a.has_z, keep = a.keep;
    const uint32_t rl = threadIdx.x & (R - 1);
    uint32_t g = threadIdx.x >> lr;
    const uint32_t row = lb * R + rl;
    const bool live = row < a.rows;
    Rec *rec = (Rec *)lds;                              // [K]
    EdgeRec *erec = (EdgeRec *)(rec + K);               // [NE][K]
    ZRec *zs = (ZRec *)(erec + NE * K);                 // [Kz]
    KeyT *red = (KeyT *)(zs + (has_z ? Kz : 0));        // [waves][min(R, 64)][2]
    const uint32_t RW = min(R, 64u);
    KeyT *X = red + (threads / 64) * RW * 2;            // [K][R] when keep
    uint32_t *cs = (uint32_t *)(X + (keep ? K << lr : 0));   // [K] configurations in class order (lookups)

    for (uint32_t c = threadIdx.x; c < K; c += threads) {
        const uint32_t at = has_z ? glb<uint16_t>(a.inv)[c] : c;
        Rec r;
        r.x = glb<KeyT>(a.Lk)[c];
        r.f = has_z ? glb<KeyT>(a.fzc)[c] : (KeyT)0;
        EdgeRec er[ME];
#pragma unroll
        for (int t = 0; t < NE; t++) {
            er[t].sig = glb<uint64_t>(a.e[t].sig_c)[c];
            er[t].f = glb<KeyT>(a.e[t].f_c)[c];
        }
        rec[at] = r;
#pragma unroll
        for (int t = 0; t < NE; t++) erec[t * K + at] = er[t];
        if (NT > 0) cs[at] = c;
    }
    if (has_z)
        for (uint32_t q = threadIdx.x; q < Kz; q += threads) {
            const uint64_t w = glb<uint64_t>(a.zs)[q];   // ClassEntry: first, count, z
            ZRec r;
            r.place = (uint32_t)w;
            r.z = (uint32_t)(w >> 32);
            r.f = glb<KeyT>(a.fzo)[r.z];
            zs[q] = r;
        }
    uint32_t d[kMaxDep];
    {
        uint32_t x = live ? row : a.rows - 1;
        for (int k = kMaxDep - 1; k >= 0; k--)
            if (k < (int)a.nR) {
                d[k] = k ? x % a.rad[k] : x;
                if (k) x /= a.rad[k];
            } else d[k] = 0;
    }
    uint64_t so[ME];
    KeyT fo[ME];
    Glb<const Val> tp[MT];
    uint32_t tsc[MT];
#pragma unroll
    for (int t = 0; t < NE; t++) {
        uint32_t w = 0;
        for (int k = 0; k < kMaxDep; k++) w = k == (int)a.e[t].dig ? d[k] : w;
        so[t] = glb<uint64_t>(a.e[t].sig_o)[w];
        fo[t] = glb<KeyT>(a.e[t].f_o)[w];
    }
#pragma unroll
    for (int t = 0; t < NT; t++) {
        uint32_t o = 0;
        for (int k = 0; k < kMaxDep; k++)
            if (k < (int)a.nR) o += d[k] * a.t[t].sd[k];
        tp[t] = glb<Val>(a.t[t].ptr) + o;
        tsc[t] = a.t[t].sc;
    }
    const uint32_t bits = a.bits, out_shift = a.out_shift, rows = a.rows;
    const Glb<Val> T = (Glb<Val>)(uintptr_t)a.T;
    const Glb<uint16_t> A = (Glb<uint16_t>)(uintptr_t)a.A;
    __syncthreads();
    if (!keep && has_z) g = __builtin_amdgcn_readfirstlane(g);   // (64 rows: a group is a wave)

    // X of the configuration at place p: its terms, then their sum
    struct Terms { Rec r; EdgeRec e[ME]; KeyT t[MT]; };
    auto fetch = [&](uint32_t p) {
        Terms v;
        if (NT > 0) {
            const uint32_t c = cs[p];
#pragma unroll
            for (int t = 0; t < NT; t++) v.t[t] = class_term<KeyT>(a.t[t].raw, bits, tp[t][(uint64_t)c * tsc[t]]);
        }
        v.r = rec[p];
#pragma unroll
        for (int t = 0; t < NE; t++) v.e[t] = erec[t * K + p];
        return v;
    };
    auto sum = [&](const Terms &v) {
        KeyT x = v.r.x;
#pragma unroll
        for (int t = 0; t < NE; t++) x = Ops::add(x, v.e[t].sig == so[t] ? (KeyT)0 : Ops::min(v.e[t].f, fo[t]));
#pragma unroll
        for (int t = 0; t < NT; t++) x = Ops::add(x, v.t[t]);
        return x;
    };
    KeyT m0 = Ops::sentinel(), m1 = Ops::sentinel();
    for (uint32_t p0 = g; p0 < K; p0 += U * G) {
        Terms v[U];
#pragma unroll
        for (int u = 0; u < U; u++) v[u] = fetch(min(p0 + u * G, K - 1));
#pragma unroll
        for (int u = 0; u < U; u++) {
            // (past the end: the last configuration once more, the same minima and store)
            const uint32_t p = min(p0 + u * G, K - 1);
            const KeyT x = sum(v[u]);
            m0 = Ops::min(m0, x);
            m1 = Ops::min(m1, Ops::add(x, v[u].r.f));
            if (keep) X[(p << lr) + rl] = x;
        }
    }
    for (uint32_t m = R; m < 64; m <<= 1) {
        m0 = Ops::min(m0, shfl_xor_key(m0, (int)m));
        m1 = Ops::min(m1, shfl_xor_key(m1, (int)m));
    }
    const uint32_t wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if (lane < RW) {
        red[(wave * RW + lane) * 2] = m0;
        red[(wave * RW + lane) * 2 + 1] = m1;
    }
    __syncthreads();
    for (uint32_t w = 0; w < threads / 64; w++) {
        m0 = Ops::min(m0, red[(w * RW + rl) * 2]);
        m1 = Ops::min(m1, red[(w * RW + rl) * 2 + 1]);
    }
    if (!live) return;
    auto put = [&](uint64_t idx, KeyT key) {
        Val v;
        uint32_t cc;
        Ops::split(key, bits, out_shift, v, cc);
        T[idx] = v;
        A[idx] = (uint16_t)cc;
    };
    if (!has_z) {
        if (g == 0) put(row, m0);
        return;
    }
    if (keep) {
        for (uint32_t q = g; q < Kz; q += G) {
            const ZRec r = zs[q];
            const uint32_t first = r.place & 0xffff, count = r.place >> 16;
            KeyT best = Ops::min(m1, Ops::add(m0, r.f));
            for (uint32_t k = 0; k < count; k++) best = Ops::min(best, X[((first + k) << lr) + rl]);
            put((uint64_t)r.z * rows + row, best);
        }
    } else {
        const uint32_t per = (Kz + G - 1) / G, q1 = min(Kz, (g + 1) * per);
        uint32_t last = ~0u;
        KeyT s = Ops::sentinel();
        for (uint32_t q = min(Kz, g * per); q < q1; q++) {
            const ZRec r = zs[q];
            const uint32_t place = __builtin_amdgcn_readfirstlane(r.place);
            if (place != last) {
                last = place;
                s = Ops::sentinel();
                for (uint32_t k = 0; k < place >> 16; k++) s = Ops::min(s, sum(fetch((place & 0xffff) + k)));
            }
            put((uint64_t)r.z * rows + row, Ops::min(s, Ops::min(m1, Ops::add(m0, r.f))));
        }
    }
}

template <typename KeyT, int NE, int NT>
__device__ __forceinline__ void class_item(const ClassArgs &a, uint32_t b, char *lds) {
    // blocks are dealt round-robin to the 8 XCDs (block counts and first blocks
    // are multiples of 8): a contiguous range of rows per XCD, so that the
    // lines two neighbouring workgroups share are completed in one L2
    const uint32_t lb = (b % 8) * (a.nblk / 8) + b / 8;
    if (lb >= (a.rows + (1u << a.lr) - 1) >> a.lr) return;   // the whole workgroup leaves together
    if (a.staged) class_item_staged<KeyT, NE, NT>(a, lb, lds);
    else class_item_small<KeyT, NE, NT>(a, lb, lds);
}

// ------------------------------------------------------------------ joint fill
// Keys moved between lanes: both halves of the 64-bit pattern.
template <int CTRL, typename KeyT> __device__ __forceinline__ KeyT dpp_key(KeyT v) {
    struct W { uint32_t lo, hi; } x = __builtin_bit_cast(W, v);
    x.lo = __builtin_amdgcn_update_dpp(x.lo, x.lo, CTRL, 0xf, 0xf, false);
    x.hi = __builtin_amdgcn_update_dpp(x.hi, x.hi, CTRL, 0xf, 0xf, false);
    return __builtin_bit_cast(KeyT, x);
}

// Minima of N = 8 or 4 keys over the wave.  Two exchange steps leave each
// row of 16 lanes with one key of every N / 4 (lane swaps between two
// registers, so no key is reduced where another will do), four steps within
// the rows finish: 42 instructions for 8 keys instead of 144.  Key k's minimum
// lands in lane 15 + 16 * (k / (N / 4)) of out[k % (N / 4)].
template <int N, typename KeyT> __device__ __forceinline__ void wave_minima(const KeyT (&v)[N], KeyT (&out)[N / 4]) {
    using Ops = KeyOps<KeyT>;
    struct W { uint32_t lo, hi; };
    KeyT w[N / 2];
#pragma unroll
    for (int k = 0; k < N / 2; k++) {
        const W a = __builtin_bit_cast(W, v[k]), b = __builtin_bit_cast(W, v[k + N / 2]);
        const auto lo = __builtin_amdgcn_permlane32_swap(a.lo, b.lo, false, false);
        const auto hi = __builtin_amdgcn_permlane32_swap(a.hi, b.hi, false, false);
        w[k] = Ops::min(__builtin_bit_cast(KeyT, W{lo[0], hi[0]}), __builtin_bit_cast(KeyT, W{lo[1], hi[1]}));
    }
#pragma unroll
    for (int k = 0; k < N / 4; k++) {
        const W a = __builtin_bit_cast(W, w[k]), b = __builtin_bit_cast(W, w[k + N / 4]);
        const auto lo = __builtin_amdgcn_permlane16_swap(a.lo, b.lo, false, false);
        const auto hi = __builtin_amdgcn_permlane16_swap(a.hi, b.hi, false, false);
        KeyT x = Ops::min(__builtin_bit_cast(KeyT, W{lo[0], hi[0]}), __builtin_bit_cast(KeyT, W{lo[1], hi[1]}));
        x = Ops::min(x, dpp_key<0x111>(x));   // row_shr 1, 2, 4, 8: lane 15 of a row ends with its minimum
        x = Ops::min(x, dpp_key<0x112>(x));
        x = Ops::min(x, dpp_key<0x114>(x));
        x = Ops::min(x, dpp_key<0x118>(x));
        out[k] = x;
    }
}

template <typename KeyT> __device__ __forceinline__ KeyT shift_key(KeyT x, int32_t s) {
    if constexpr (std::is_same<KeyT, double>::value) return x * __builtin_ldexp(1.0, s);
    else return s >= 0 ? x << s : x >> -s;
}

// Class ids of one joint shape: one workgroup, a thread per configuration
// (at most kJointMaxK).
struct JointTabLds {
    uint16_t rank[4][kJointMaxK];   // by place of the four class orders: number of the class there
    uint16_t wave_sum[4][16];
    JointIdJ id[2][kJointMaxK];     // both sides: own, other, y, both
    uint16_t place[kJointMaxK];     // v_i: place by (y class, own class)
};
__device__ __forceinline__ void joint_table_item(const DevJointTab &jt, const DevClassTab *__restrict__ tabs,
                                                 char *__restrict__ ws, JointTabLds &lds) {
    const uint32_t t = threadIdx.x, lane = t & 63, wave = t >> 6;
    auto place0 = [&](int k, uint32_t c) { return ((const uint16_t *)(ws + tabs[jt.tab[k]].first_off))[c]; };
    auto perm = [&](int k, uint32_t p) { return ((const uint16_t *)(ws + tabs[jt.tab[k]].perm_off))[p]; };
    auto zr = [&](int k, uint32_t z) { return ((const uint32_t *)(ws + tabs[jt.tab[k]].zr_off))[z]; };
    // number the classes of each order: a place starts a class when it is the
    // first place of the configuration there
    bool starts[4];
    for (int k = 0; k < 4; k++) {
        const bool in = jt.tab[k] >= 0 && t < tabs[jt.tab[k]].K;
        starts[k] = in && place0(k, perm(k, t)) == t;
        const uint64_t m = __ballot(starts[k]);
        if (lane == 0) lds.wave_sum[k][wave] = (uint16_t)__popcll(m);
        // (classes started up to and including this place, within the wave)
        lds.rank[k][t] = (uint16_t)__popcll(m & (~0ull >> (63 - lane)));
    }
    __syncthreads();
    for (int k = 0; k < 4; k++) {
        uint32_t s = 0;
        for (uint32_t w = 0; w < wave; w++) s += lds.wave_sum[k][w];
        const uint32_t r = lds.rank[k][t] + s - 1;
        lds.rank[k][t] = (uint16_t)r;
        const int at = k == 3 ? 0 : k == 0 ? 1 : k == 1 ? 2 : -1;   // i to j, i to y, j to y
        if (at >= 0 && jt.tab[k] >= 0) {
            uint16_t *out = (uint16_t *)(ws + jt.off_start[at]);
            if (starts[k]) out[r] = (uint16_t)t;
            if (t + 1 == tabs[jt.tab[k]].K) out[r + 1] = (uint16_t)(t + 1);
        }
    }
    __syncthreads();
    // side 0: v_i (orders 3: to j, 0: to y), side 1: v_j (orders 2: to i, 1: to y)
    const bool has_e = jt.tab[0] >= 0;
    for (int sd = 0; sd < 2; sd++) {
        const int o = sd ? 2 : 3, oo = sd ? 3 : 2, y = sd ? 1 : 0;
        if (t >= tabs[jt.tab[o]].K) continue;
        JointIdJ id;
        id.own = lds.rank[o][place0(o, t)];
        const uint32_t z = zr(oo, t);
        id.other = z >> 16 ? lds.rank[oo][z & 0xffff] : (uint16_t)kNoClass;
        id.y = jt.tab[y] >= 0 ? lds.rank[y][place0(y, t)] : (uint16_t)0;
        id.both = (uint16_t)t;
        lds.id[sd][t] = id;
    }
    __syncthreads();
    for (int sd = 0; sd < 2; sd++) {
        const int o = sd ? 2 : 3, y = sd ? 1 : 0;
        const uint32_t K = tabs[jt.tab[o]].K;
        if (t >= K || !has_e) continue;
        // within its class to y: the lowest configuration that shares the
        // other class, and how many come before it by (other class, index)
        const JointIdJ id = lds.id[sd][t];
        uint32_t best = t, before = 0;
        for (uint32_t p = place0(y, t); p < K; p++) {
            const uint32_t c = perm(y, p);
            const JointIdJ q = lds.id[sd][c];
            if (q.y != id.y) break;
            if (q.own == id.own && c < best) best = c;
            before += q.own < id.own || (q.own == id.own && c < t);
        }
        lds.id[sd][t].both = (uint16_t)best;
        if (sd == 0) lds.place[t] = (uint16_t)(place0(y, t) + before);
    }
    __syncthreads();
    if (t < tabs[jt.tab[3]].K)
        ((JointIdI *)(ws + jt.off_i))[t] =
            JointIdI{((const uint16_t *)(ws + tabs[jt.tab[3]].inv_off))[t], has_e ? lds.place[t] : (uint16_t)0,
                     lds.id[0][t].other, 0};
    if (t < tabs[jt.tab[2]].K) {
        ((JointIdJ *)(ws + jt.off_j))[t] = lds.id[1][t];
        ((uint16_t *)(ws + jt.off_jown))[t] = lds.id[1][perm(1, t)].other;
    }
    if (t >= tabs[jt.tab[1]].Kz) return;
    JointY r;
    const uint32_t zj = zr(1, t), zi = has_e ? zr(0, t) : 0;
    r.i = zi >> 16 ? lds.rank[0][zi & 0xffff] : (uint16_t)kNoClass;
    r.j = zj >> 16 ? lds.rank[1][zj & 0xffff] : (uint16_t)kNoClass;
    r.first = r.count = 0;
    r.pj = (uint16_t)kNoClass;
    r.pad[0] = r.pad[1] = r.pad[2] = 0;
    for (uint32_t k = 0; k < zi >> 16 && r.pj == kNoClass; k++) {
        const uint32_t c = perm(0, (zi & 0xffff) + k), want = lds.id[0][c].other;
        for (uint32_t l = 0; l < zj >> 16 && want != kNoClass; l++) {
            const uint32_t cp = perm(1, (zj & 0xffff) + l);
            if (lds.id[1][cp].own != want) continue;
            r.pj = lds.id[1][cp].both;
            const uint32_t lowest = lds.id[0][c].both;
            r.first = lds.place[lowest];
            for (uint32_t m = 0; m < zi >> 16; m++) r.count += lds.id[0][perm(0, (zi & 0xffff) + m)].both == lowest;
            break;
        }
    }
    ((JointY *)(ws + jt.off_y))[t] = r;
}

// XI or XJ of configuration c (its row-independent data in sg, ef) at digits d.
template <typename KeyT>
__device__ __forceinline__ KeyT joint_sum(const JointSide &s, uint32_t nR, uint32_t c, KeyT lk,
                                          const uint64_t (&sg)[kJointTerms], const KeyT (&ef)[kJointTerms],
                                          const uint32_t (&d)[kMaxDep]) {
    using Ops = KeyOps<KeyT>;
    using Val = typename Ops::Val;
    KeyT v = lk;
#pragma unroll
    for (int t = 0; t < (int)kJointTerms; t++)
        if (t < (int)s.nt) {
            uint64_t o = (uint64_t)c * s.t[t].sc;
            for (int k = 0; k < kMaxDep; k++)
                if (k < (int)nR) o += (uint64_t)d[k] * s.t[t].sd[k];
            v = Ops::add(v, __builtin_bit_cast(KeyT, glb<Val>(s.t[t].ptr)[o]));
        }
#pragma unroll
    for (int t = 0; t < (int)kJointTerms; t++)
        if (t < (int)s.ne) {
            uint32_t w = 0;
            for (int k = 0; k < kMaxDep; k++) w = k == (int)s.e[t].dig ? d[k] : w;
            const uint64_t so = glb<uint64_t>(s.e[t].sig_o)[w];
            v = Ops::add(v, sg[t] == so ? (KeyT)0 : Ops::min(ef[t], glb<KeyT>(s.e[t].f_o)[w]));
        }
    return v;
}

// Non-negative keys order like their bit patterns: minima in LDS by 64-bit
// integer atomics.  An untouched one (all ones) reads as the sentinel.
template <typename KeyT> __device__ __forceinline__ void lds_min(uint64_t *p, KeyT v) {
    atomicMin((unsigned long long *)p, __builtin_bit_cast(unsigned long long, v));
}
template <typename KeyT> __device__ __forceinline__ KeyT lds_key(const uint64_t *p) {
    const uint64_t v = *p;
    if constexpr (std::is_same<KeyT, double>::value)
        return v == ~0ull ? KeyOps<double>::sentinel() : __builtin_bit_cast(double, v);
    else return v;
}

// Half fill: workgroup b takes upper indices b, b + hblk, ...; configurations
// over the threads, U per thread.
template <typename KeyT, int U>
__device__ __forceinline__ void half_item(const JointArgs &a, uint32_t b, char *lds) {
    using Ops = KeyOps<KeyT>;
    constexpr int M = (int)kJointTerms;
    const uint32_t tid = threadIdx.x, threads = blockDim.x, lane = tid & 63;
    const uint32_t Ki = a.s[0].K, Kj = a.s[1].K, Ky = a.Ky;
    uint64_t *sl = (uint64_t *)lds, *mJ = sl + 16, *mJy = mJ + a.oj, *yJ = mJy + a.oj, *yJf = yJ + a.yj, *bJ = yJf + a.yj;
    const uint32_t nslots = 16 + 2 * a.oj + 2 * a.yj + Kj;
    const int32_t shift = a.s[1].shift;
    const uint64_t stride = 2 * (uint64_t)Ki + Kj + 3 * (uint64_t)Ky;
    for (uint32_t up = b; up < a.upper; up += a.hblk) {
        __syncthreads();
        for (uint32_t k = tid; k < nslots; k += threads) sl[k] = ~0ull;
        uint32_t d[kMaxDep];
        uint32_t x = up * a.lower;
        for (int k = kMaxDep - 1; k >= 0; k--)
            if (k < (int)a.nR) { d[k] = k ? x % a.rad[k] : x; if (k) x /= a.rad[k]; } else d[k] = 0;
        KeyT xj[U], f[U], g[U], m[4] = {Ops::sentinel(), Ops::sentinel(), Ops::sentinel(), Ops::sentinel()};
        JointIdJ id[U];
#pragma unroll
        for (int u = 0; u < U; u++) {
            const uint32_t c = min(tid + u * threads, Kj - 1);
            uint64_t sg[M];
            KeyT ef[M];
#pragma unroll
            for (int t = 0; t < M; t++) {
                sg[t] = t < (int)a.s[1].ne ? glb<uint64_t>(a.s[1].e[t].sig_c)[c] : 0;
                ef[t] = t < (int)a.s[1].ne ? glb<KeyT>(a.s[1].e[t].f_c)[c] : (KeyT)0;
            }
            id[u] = __builtin_bit_cast(JointIdJ, glb<uint64_t>(a.ij)[c]);
            f[u] = shift_key(glb<KeyT>(a.fj_o)[c], shift);
            g[u] = shift_key(glb<KeyT>(a.fj_y)[c], shift);
            // without its configuration bits, in v_i's key space
            xj[u] = shift_key((KeyT)(joint_sum<KeyT>(a.s[1], a.nR, c, glb<KeyT>(a.s[1].Lk)[c], sg, ef, d) - (KeyT)c), shift);
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < U; u++) {
            const KeyT xf = Ops::add(xj[u], f[u]), xy = Ops::add(xj[u], g[u]);
            m[0] = Ops::min(m[0], xj[u]);
            m[1] = Ops::min(m[1], xf);
            m[2] = Ops::min(m[2], xy);
            m[3] = Ops::min(m[3], Ops::add(xy, f[u]));
            if (tid + u * threads >= Kj) continue;
            lds_min(&mJ[id[u].own], xj[u]);
            lds_min(&mJy[id[u].own], xy);
            lds_min(&yJ[id[u].y], xj[u]);
            lds_min(&yJf[id[u].y], xf);
            lds_min(&bJ[id[u].both], xj[u]);
        }
        KeyT r[1];
        wave_minima<4>(m, r);
        if ((lane & 15) == 15) lds_min(&sl[lane >> 4], r[0]);
        __syncthreads();
        const KeyT s0 = lds_key<KeyT>(&sl[0]), s1 = lds_key<KeyT>(&sl[1]), s2 = lds_key<KeyT>(&sl[2]),
                   s3 = lds_key<KeyT>(&sl[3]);
        const Glb<KeyT> out = (Glb<KeyT>)(uintptr_t)a.half + up * stride;
#pragma unroll
        for (int u = 0; u < U; u++) {
            const uint32_t c = tid + u * threads;
            if (c < Ki) {
                const JointIdI ii = __builtin_bit_cast(JointIdI, glb<uint64_t>(a.ii)[c]);
                const KeyT fi = shift_key(glb<KeyT>(a.fi_o)[c], shift);
                KeyT j0 = Ops::min(s1, Ops::add(fi, s0)), j1 = Ops::min(s3, Ops::add(fi, s2));
                if (ii.other != kNoClass) {
                    j0 = Ops::min(j0, lds_key<KeyT>(&mJ[ii.other]));
                    j1 = Ops::min(j1, lds_key<KeyT>(&mJy[ii.other]));
                }
                out[c] = j0;
                out[Ki + c] = j1;
            }
            if (c < Kj) out[2 * (uint64_t)Ki + glb<uint16_t>(a.jplace)[c]] = xj[u];
            if (c < Ky) {
                const JointY y = a.y[c];
                const bool in = y.j != kNoClass;
                const Glb<KeyT> oy = out + 2 * (uint64_t)Ki + Kj + c;
                oy[0] = in ? lds_key<KeyT>(&yJ[y.j]) : Ops::sentinel();
                oy[Ky] = in ? lds_key<KeyT>(&yJf[y.j]) : Ops::sentinel();
                oy[2 * (uint64_t)Ky] = y.pj != kNoClass ? lds_key<KeyT>(&bJ[y.pj]) : Ops::sentinel();
            }
        }
    }
}

// Joint fill: workgroup b takes one upper index and every seg-th of its lower
// ones, one row at a time; configurations over the threads, U per thread, so
// a table row is stored contiguously and everything that does not depend on
// the lower digits stays in registers and LDS.  XI goes to LDS in class order,
// so a class's minimum is a thread's walk over a few neighbouring values;
// three barriers per row (XI and its minima; class minima; those of XJ + I),
// then the row's entries.
//
// Bound by none of the units: by the chain of steps in a row and their
// barriers.  38 808 rows of 462 configurations (316 us under the counters):
// 2430 VALU and 456 LDS wave instructions per row, VALU busy for 52% of its
// cycles, LDS for 36% (a third of these bank conflicts), waves waiting for 64%
// of theirs with 20 of them per CU.  148 393 rows of 731: 5140 and 1150, 45%,
// 34%, 74% with 22 per CU; stores 0.38 TB/s.  The walks over classes of 1 to 24
// members leave most lanes of their waves idle.  On small vertices by the
// latency of the steps alone.
//
// Measured on the Transformer at p = 64: a cross-attention score vertex (7056
// rows, 3.3e6 entries of 462 configurations) 68 us against 167 + 26 us for the
// dense fill and its prep; the fourth decoder's key/value projection (38808
// rows) 311 us against 613 + 162 us -- and the five tables these two kinds read,
// 180 MB each, are not formed at all (level 0: 244 -> 21 us).  140 registers
// instead of 80 (one workgroup per CU instead of three) took 131 and 654 us;
// class members read four at a time, the last one repeated, 80 and 364 us.
template <typename KeyT, int U, bool HASE>
__device__ __forceinline__ void joint_item(const JointArgs &a, uint32_t b, char *lds) {
    using Ops = KeyOps<KeyT>;
    using Val = typename Ops::Val;
    constexpr int M = (int)kJointTerms;
    const uint32_t tid = threadIdx.x, threads = blockDim.x, lane = tid & 63;
    const uint32_t Ki = a.s[0].K, Kj = a.s[1].K, Ky = a.Ky, oi = a.oi, yi = a.yi, yj = a.yj;
    // XCD-contiguous ranges of workgroups: the segments of one upper index
    // read neighbouring lines of the lookups
    const uint32_t w = (b % 8) * (a.nblk / 8) + b / 8, up = w / a.seg;
    if (up >= a.upper) return;   // the whole workgroup leaves together
    uint64_t *slots = (uint64_t *)lds;                       // [2][16] row minima, by row parity
    KeyT *XO = (KeyT *)(slots + 32);                         // XI by own class
    KeyT *CI0 = XO + Ki, *VV0 = CI0 + oi, *XJ = VV0 + yj;    // minima of XI by own class; of XJ + that by y class
    KeyT *XY = XJ + Kj;                                      // [2] XI by y class, by row parity
    KeyT *PA = XY + (HASE ? 2 * Ki : 0), *PB = PA + (HASE ? Ki : 0);      // P0, P1 by y class
    KeyT *FO = PB + (HASE ? Ki : 0), *FY = FO + (HASE ? Ki : 0);          // f to y by own class, f to v_j by y class
    KeyT *CI1 = FY + (HASE ? Ki : 0), *Q0 = CI1 + (HASE ? oi : 0), *Q1 = Q0 + (HASE ? yi : 0);
    KeyT *A0 = Q1 + (HASE ? yi : 0), *A1 = A0 + (HASE ? yi : 0), *VV1 = A1 + (HASE ? yi : 0);
    uint16_t *so = (uint16_t *)(VV1 + (HASE ? yj : 0)), *sy = so + oi + 1, *sj = sy + yi + 1, *jown = sj + yj + 1;

    const int32_t shift = a.s[1].shift;
    const Glb<const KeyT> half = glb<KeyT>(a.half) + up * (2 * (uint64_t)Ki + Kj + 3 * (uint64_t)Ky);
    KeyT lk[U], fo[U], fy[U], j0[U], j1[U], ef[U][M];
    uint64_t sg[U][M];
    uint32_t po[U], py[U];
    KeyT hI[U], hJ[U], b0[U], b1[U], bp[U];
    JointY dy[U];
#pragma unroll
    for (int u = 0; u < U; u++) {
        const uint32_t c = tid + u * threads, ci = min(c, Ki - 1), y = min(c, Ky - 1);
        lk[u] = glb<KeyT>(a.s[0].Lk)[ci];
        fo[u] = shift_key(glb<KeyT>(a.fi_o)[ci], shift);   // (the edge between the two is in v_j's keys)
        fy[u] = HASE ? glb<KeyT>(a.fi_y)[ci] : (KeyT)0;
        j0[u] = half[ci];
        j1[u] = half[Ki + ci];
        const JointIdI id = __builtin_bit_cast(JointIdI, glb<uint64_t>(a.ii)[ci]);
        po[u] = id.own;
        py[u] = id.yplace;
#pragma unroll
        for (int t = 0; t < M; t++) {
            sg[u][t] = t < (int)a.s[0].ne ? glb<uint64_t>(a.s[0].e[t].sig_c)[ci] : 0;
            ef[u][t] = t < (int)a.s[0].ne ? glb<KeyT>(a.s[0].e[t].f_c)[ci] : (KeyT)0;
        }
        hJ[u] = shift_key(glb<KeyT>(a.fj_yy)[y], shift);
        hI[u] = HASE ? glb<KeyT>(a.fi_yy)[y] : (KeyT)0;
        const Glb<const KeyT> hy = half + 2 * (uint64_t)Ki + Kj + y;
        b0[u] = hy[0];
        b1[u] = hy[Ky];
        bp[u] = hy[2 * (uint64_t)Ky];
        dy[u] = a.y[y];
        if (c < Ki && HASE) {
            FO[po[u]] = fy[u];
            FY[py[u]] = fo[u];
        }
        if (c < Kj) {
            XJ[c] = half[2 * (uint64_t)Ki + c];
            jown[c] = glb<uint16_t>(a.jown)[c];
        }
    }
    for (uint32_t k = tid; k <= oi; k += threads) so[k] = glb<uint16_t>(a.start_o)[k];
    if (HASE)
        for (uint32_t k = tid; k <= yi; k += threads) sy[k] = glb<uint16_t>(a.start_yi)[k];
    for (uint32_t k = tid; k <= yj; k += threads) sj[k] = glb<uint16_t>(a.start_yj)[k];
    if (tid < 32) slots[tid] = ~0ull;
    const uint32_t bits = a.bits, out_shift = a.out_shift;
    const Glb<Val> T = (Glb<Val>)(uintptr_t)a.T;
    const Glb<uint16_t> A = (Glb<uint16_t>)(uintptr_t)a.A;
    uint32_t parity = 0;
    auto xi_of = [&](uint32_t row, KeyT (&xi)[U]) {
        uint32_t d[kMaxDep];
        uint32_t x = row;
        for (int k = kMaxDep - 1; k >= 0; k--)
            if (k < (int)a.nR) { d[k] = k ? x % a.rad[k] : x; if (k) x /= a.rad[k]; } else d[k] = 0;
#pragma unroll
        for (int u = 0; u < U; u++)   // (past the end: the last configuration again)
            xi[u] = joint_sum<KeyT>(a.s[0], a.nR, min(tid + u * threads, Ki - 1), lk[u], sg[u], ef[u], d);
    };
    KeyT xi[U];
    if (w % a.seg < a.lower) xi_of(up * a.lower + w % a.seg, xi);
    __syncthreads();
    for (uint32_t lowi = w % a.seg; lowi < a.lower; lowi += a.seg, parity ^= 1) {
        const uint32_t row = up * a.lower + lowi;
        uint64_t *sl = slots + 16 * parity;
        KeyT *XYp = XY + (HASE ? parity * Ki : 0);
        KeyT m[8];
#pragma unroll
        for (int k = 0; k < 8; k++) m[k] = Ops::sentinel();
#pragma unroll
        for (int u = 0; u < U; u++) {
            const KeyT p0 = Ops::add(xi[u], j0[u]), p1 = Ops::add(xi[u], j1[u]);
            m[0] = Ops::min(m[0], xi[u]);
            m[1] = Ops::min(m[1], Ops::add(xi[u], fo[u]));
            m[2] = Ops::min(m[2], p0);
            m[3] = Ops::min(m[3], p1);
            XO[po[u]] = xi[u];
            if (HASE) {
                const KeyT xy = Ops::add(xi[u], fy[u]);
                m[4] = Ops::min(m[4], xy);
                m[5] = Ops::min(m[5], Ops::add(xy, fo[u]));
                m[6] = Ops::min(m[6], Ops::add(p0, fy[u]));
                m[7] = Ops::min(m[7], Ops::add(p1, fy[u]));
                XYp[py[u]] = xi[u];
                PA[py[u]] = p0;
                PB[py[u]] = p1;
            }
        }
        if (HASE) {
            KeyT r[2];
            wave_minima<8>(m, r);
            if ((lane & 15) == 15) {
                lds_min(&sl[2 * (lane >> 4)], r[0]);
                lds_min(&sl[2 * (lane >> 4) + 1], r[1]);
            }
        } else {
            KeyT r[1], m4[4] = {m[0], m[1], m[2], m[3]};
            wave_minima<4>(m4, r);
            if ((lane & 15) == 15) lds_min(&sl[lane >> 4], r[0]);
        }
        __syncthreads();
        // the next row's minima (their last readers are past the barrier) and XI
        if (tid < 16) slots[16 * (parity ^ 1) + tid] = ~0ull;
        if (lowi + a.seg < a.lower) xi_of(row + a.seg, xi);
        // class minima: a thread per class of either order
        for (uint32_t k = tid; k < oi + (HASE ? yi : 0); k += threads) {
            if (k < oi) {
                KeyT v = Ops::sentinel(), v1 = Ops::sentinel();
                for (uint32_t p = so[k]; p < so[k + 1]; p++) {
                    const KeyT x = XO[p];
                    v = Ops::min(v, x);
                    if (HASE) v1 = Ops::min(v1, Ops::add(x, FO[p]));
                }
                CI0[k] = v;
                if (HASE) CI1[k] = v1;
            } else if (HASE) {
                KeyT q0 = Ops::sentinel(), q1 = Ops::sentinel(), v = Ops::sentinel(), v1 = Ops::sentinel();
                for (uint32_t p = sy[k - oi]; p < sy[k - oi + 1]; p++) {
                    const KeyT x = XYp[p];
                    v = Ops::min(v, x);
                    v1 = Ops::min(v1, Ops::add(x, FY[p]));
                    q0 = Ops::min(q0, PA[p]);
                    q1 = Ops::min(q1, PB[p]);
                }
                Q0[k - oi] = q0;
                Q1[k - oi] = q1;
                A0[k - oi] = v;
                A1[k - oi] = v1;
            }
        }
        __syncthreads();
        for (uint32_t k = tid; k < yj; k += threads) {
            KeyT v = Ops::sentinel(), v1 = Ops::sentinel();
            for (uint32_t p = sj[k]; p < sj[k + 1]; p++) {
                const uint32_t o = jown[p];
                if (o == kNoClass) continue;
                const KeyT x = XJ[p];
                v = Ops::min(v, Ops::add(x, CI0[o]));
                if (HASE) v1 = Ops::min(v1, Ops::add(x, CI1[o]));
            }
            VV0[k] = v;
            if (HASE) VV1[k] = v1;
        }
        __syncthreads();
        KeyT s[8];
#pragma unroll
        for (int k = 0; k < (HASE ? 8 : 4); k++) s[k] = lds_key<KeyT>(&sl[k]);
#pragma unroll
        for (int u = 0; u < U; u++) {
            const uint32_t y = tid + u * threads;
            if (y >= Ky) break;
            KeyT best = Ops::min(Ops::add(s[2], hJ[u]), s[3]);
            const bool ni = HASE && dy[u].i != kNoClass, nj = dy[u].j != kNoClass;
            if (HASE) best = Ops::min(Ops::add(best, hI[u]), Ops::min(Ops::add(s[6], hJ[u]), s[7]));
            if (nj) {   // c' in y's class: XJ + I0, XJ + I1
                KeyT v = Ops::min(VV0[dy[u].j], Ops::min(Ops::add(b1[u], s[0]), Ops::add(b0[u], s[1])));
                if (HASE) v = Ops::add(v, hI[u]);
                best = Ops::min(best, v);
                if (HASE)
                    best = Ops::min(best, Ops::min(VV1[dy[u].j], Ops::min(Ops::add(b1[u], s[4]), Ops::add(b0[u], s[5]))));
            }
            if (ni) {
                best = Ops::min(best, Ops::min(Ops::add(Q0[dy[u].i], hJ[u]), Q1[dy[u].i]));
                if (nj) {   // both in y's classes: t(c', c) one of the f, or 0
                    best = Ops::min(best, Ops::min(Ops::add(A0[dy[u].i], b1[u]), Ops::add(A1[dy[u].i], b0[u])));
                    for (uint32_t k = 0; k < dy[u].count; k++)
                        best = Ops::min(best, Ops::add(XYp[dy[u].first + k], bp[u]));
                }
            }
            Val v;
            uint32_t cc;
            Ops::split(best, bits, out_shift, v, cc);
            const uint64_t idx = (uint64_t)row * Ky + y;
            T[idx] = v;
            A[idx] = (uint16_t)cc;
        }
    }
}

// ------------------------------------------------------------------ exchange fill
// What a class without configurations reads as: past every key, and summed
// with two of them still no more than 2^63.
template <typename KeyT> __device__ __forceinline__ KeyT exch_none() {
    if constexpr (std::is_same<KeyT, double>::value) return KeyOps<double>::sentinel();
    else return (KeyT)1 << 62;
}

// Half fill of an exchange: workgroup c evaluates A' = A[c][x] + L_i[x] over all
// x and its minima over the classes to y and to z (in LDS, by the class's first
// place), then what the fill reads by y and by z.  The lowest x of a pair of
// classes holds their common minimum.  Bound by latency (a few memory round
// trips, Kj workgroups).
template <typename KeyT>
__device__ __forceinline__ void exch_half_item(const ExchArgs &a, uint32_t c, char *lds) {
    using Ops = KeyOps<KeyT>;
    using Val = typename Ops::Val;
    const uint32_t tid = threadIdx.x, lane = tid & 63, Ki = a.Ki, Ky = a.Ky, Kz = a.Kz;
    uint64_t *sl = (uint64_t *)lds, *P1 = sl + 4, *P2 = P1 + Ki, *Q1 = P2 + Ki, *Q2 = Q1 + Ki, *I = Q2 + Ki;
    uint16_t *pm = (uint16_t *)(I + Ki), *c1 = pm + Ki, *c2 = c1 + Ki;
    const Glb<KeyT> out = (Glb<KeyT>)(uintptr_t)a.half + c * (3 * (uint64_t)a.Kyp + 3 * (uint64_t)Kz + Ki);
    auto look = [&](int k, uint32_t d) -> KeyT {
        const Val v = glb<Val>(a.l[k].ptr)[(uint64_t)c * a.l[k].sc + (uint64_t)d * a.l[k].sd];
        return shift_key(__builtin_bit_cast(KeyT, v), a.shift);
    };
    for (uint32_t k = tid; k < 4 + 5 * Ki; k += blockDim.x) sl[k] = ~0ull;
    for (uint32_t x = tid; x < Ki; x += blockDim.x) {
        pm[x] = glb<uint16_t>(a.perm1)[x];
        c1[x] = glb<uint16_t>(a.first1)[x];
        c2[x] = glb<uint16_t>(a.first2)[x];
    }
    __syncthreads();
    KeyT m[4] = {Ops::sentinel(), Ops::sentinel(), Ops::sentinel(), Ops::sentinel()};
    for (uint32_t x = tid; x < Ki; x += blockDim.x) {
        const KeyT v = Ops::add(glb<KeyT>(a.Li)[x], look(0, x)), f1 = glb<KeyT>(a.f1x)[x], f2 = glb<KeyT>(a.f2x)[x];
        const KeyT v1 = Ops::add(v, f1), v2 = Ops::add(v, f2);
        m[0] = Ops::min(m[0], v);
        m[1] = Ops::min(m[1], v1);
        m[2] = Ops::min(m[2], v2);
        m[3] = Ops::min(m[3], Ops::add(v1, f2));
        lds_min(&P1[c1[x]], v);
        lds_min(&P2[c1[x]], v2);
        lds_min(&Q1[c2[x]], v);
        lds_min(&Q2[c2[x]], v1);
        uint32_t p = c1[x];   // (ends at x itself at the latest)
        while (c2[pm[p]] != c2[x]) p++;
        lds_min(&I[pm[p]], v);
    }
    KeyT r[1];
    wave_minima<4>(m, r);
    if ((lane & 15) == 15) lds_min(&sl[lane >> 4], r[0]);
    __syncthreads();
    const KeyT s0 = lds_key<KeyT>(&sl[0]), s1 = lds_key<KeyT>(&sl[1]), s2 = lds_key<KeyT>(&sl[2]),
               s3 = lds_key<KeyT>(&sl[3]);
    const KeyT lj = shift_key((KeyT)(glb<KeyT>(a.Lj)[c] - (KeyT)c), a.shift);
    for (uint32_t y = tid; y < a.Kyp; y += blockDim.x) {
        const uint32_t w = min(y, Ky - 1), q = glb<uint32_t>(a.zr1)[w];
        const KeyT f = glb<KeyT>(a.f1y)[w], b = Ops::add(lj, look(1, w));
        KeyT u = Ops::min(Ops::add(s0, f), s1), v = Ops::min(Ops::add(s2, f), s3);
        if (q >> 16) {
            u = Ops::min(u, lds_key<KeyT>(&P1[q & 0xffff]));
            v = Ops::min(v, lds_key<KeyT>(&P2[q & 0xffff]));
        }
        out[y] = Ops::add(u, b);
        out[a.Kyp + y] = Ops::add(v, b);
        out[2 * (uint64_t)a.Kyp + y] = b;
    }
    const Glb<KeyT> oz = out + 3 * (uint64_t)a.Kyp;
    for (uint32_t z = tid; z < Kz; z += blockDim.x) {
        const uint32_t q = glb<uint32_t>(a.zr2)[z];
        const KeyT v = look(2, z);
        oz[z] = v;
        oz[Kz + z] = q >> 16 ? Ops::add(v, lds_key<KeyT>(&Q1[q & 0xffff])) : exch_none<KeyT>();
        oz[2 * (uint64_t)Kz + z] = q >> 16 ? Ops::add(v, lds_key<KeyT>(&Q2[q & 0xffff])) : exch_none<KeyT>();
    }
    for (uint32_t x = tid; x < Ki; x += blockDim.x)
        oz[3 * (uint64_t)Kz + x] = I[x] == ~0ull ? exch_none<KeyT>() : lds_key<KeyT>(&I[x]);
}

struct ExchLds {
    uint32_t rep[kExchCols][64];       // lowest x in the classes of y and z, or kNoClass
    uint64_t best[kExchCols][kExchCols][64];   // by wave, y, z
};

// Exchange fill: a workgroup takes kExchCols y's and 64 z's, one z per lane;
// its four waves take every fourth c (so that even a table of 462 x 462 entries
// has four waves per SIMD) and meet in LDS.  What depends on y is uniform over
// a wave and comes through scalar loads.  All loads of two c's are in flight
// together (branches around the few (y, z) with an x in both classes kept them
// apart: 42 us).  K = 84, 462, 462, 462: 25 us after a half
// fill of 9.5 us, against 652 us for the dense fill with the reader's minimum
// in its epilogue and its prep; K = 203, 731, 731, 731: 102 + 13 us against
// 5158 us and a generic fill of 1156 us that reads the 3.1 GB table back.
template <typename KeyT>
__device__ __forceinline__ void exch_item(const ExchArgs &a, uint32_t b, ExchLds &lds) {
    using Ops = KeyOps<KeyT>;
    using Val = typename Ops::Val;
    constexpr int Y = (int)kExchCols;
    const uint32_t lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t nz = (a.Kz + 63) / 64, y0 = b / nz * Y, z = b % nz * 64 + lane, zc = min(z, a.Kz - 1);
    // one y per wave: the lowest x of its class whose class to z is the lane's
    {
        const uint32_t y = min(y0 + wave, a.Ky - 1), q = glb<uint32_t>(a.zr1)[y], qz = glb<uint32_t>(a.zr2)[zc];
        uint32_t rep = kNoClass;
        for (uint32_t p0 = 0; p0 < q >> 16; p0 += 64) {
            const uint32_t n = min(64u, (q >> 16) - p0);
            const uint32_t x = glb<uint16_t>(a.perm1)[(q & 0xffff) + p0 + min(lane, n - 1)];
            const uint32_t cl = glb<uint16_t>(a.first2)[x];
            for (uint32_t k = 0; k < n; k++) {
                const uint32_t xk = __builtin_amdgcn_readlane(x, k), ck = __builtin_amdgcn_readlane(cl, k);
                if (rep == kNoClass && qz >> 16 && ck == (qz & 0xffff)) rep = xk;
            }
        }
        lds.rep[wave][lane] = rep;
    }
    __syncthreads();
    uint32_t rep[Y], at[Y];
#pragma unroll
    for (int k = 0; k < Y; k++) {
        rep[k] = lds.rep[k][lane];
        at[k] = min(rep[k], a.Ki - 1);
    }
    KeyT t1[Y], t2[Y], t3[Y], t5[Y];
#pragma unroll
    for (int k = 0; k < Y; k++) t1[k] = t2[k] = t3[k] = t5[k] = Ops::sentinel();
    const uint64_t pitch = 3 * (uint64_t)a.Kyp + 3 * (uint64_t)a.Kz + a.Ki;
    const KeyT *const half = (const KeyT *)a.half;
    constexpr int U = 2;   // c's in flight
    for (uint32_t c = wave; c < a.Kj; c += U * Y) {
        KeyT C[U], g[U], d[U], x[U][Y], h[U][3][Y];
#pragma unroll
        for (int u = 0; u < U; u++) {   // (past the end: the wave's first again)
            const uint64_t cu = c + u * Y < a.Kj ? c + u * Y : c;
            const Glb<const KeyT> hz = glb<KeyT>(half + cu * pitch + 3 * (uint64_t)a.Kyp);
            C[u] = hz[zc];
            g[u] = hz[a.Kz + zc];
            d[u] = hz[2 * (uint64_t)a.Kz + zc];
#pragma unroll
            for (int k = 0; k < Y; k++) x[u][k] = hz[3 * (uint64_t)a.Kz + at[k]];
            const auto hy = (const __attribute__((address_space(4))) KeyT *)(uintptr_t)(half + cu * pitch + y0);
#pragma unroll
            for (int q = 0; q < 3; q++)
#pragma unroll
                for (int k = 0; k < Y; k++) h[u][q][k] = hy[(uint64_t)q * a.Kyp + k];
        }
#pragma unroll
        for (int u = 0; u < U; u++)
#pragma unroll
            for (int k = 0; k < Y; k++) {
                t1[k] = Ops::min(t1[k], Ops::add(h[u][0][k], C[u]));
                t2[k] = Ops::min(t2[k], Ops::min(Ops::add(h[u][1][k], C[u]), Ops::add(h[u][2][k], d[u])));
                t3[k] = Ops::min(t3[k], Ops::add(h[u][2][k], g[u]));
                t5[k] = Ops::min(t5[k], Ops::add(Ops::add(h[u][2][k], C[u]), x[u][k]));
            }
    }
    const KeyT fz = glb<KeyT>(a.f2z)[zc];
#pragma unroll
    for (int k = 0; k < Y; k++) {
        const KeyT fy = glb<KeyT>(a.f1y)[min(y0 + k, a.Ky - 1)];
        // (a wave without a c holds sentinels only)
        KeyT v = wave < a.Kj ? Ops::min(t2[k], Ops::min(Ops::add(t1[k], fz), Ops::add(t3[k], fy))) : Ops::sentinel();
        if (rep[k] != kNoClass) v = Ops::min(v, t5[k]);
        lds.best[wave][k][lane] = __builtin_bit_cast(uint64_t, v);
    }
    __syncthreads();
    const uint32_t y = y0 + wave;
    if (y >= a.Ky || z >= a.Kz) return;
    KeyT best = Ops::sentinel();
#pragma unroll
    for (int w = 0; w < Y; w++) best = Ops::min(best, __builtin_bit_cast(KeyT, lds.best[w][wave][lane]));
    Val v;
    uint32_t x;
    Ops::split(best, a.bits, a.out_shift, v, x);
    const uint64_t idx = (uint64_t)y * a.Kz + z;
    ((Glb<Val>)(uintptr_t)a.T)[idx] = v;
    ((Glb<uint16_t>)(uintptr_t)a.A)[idx] = (uint16_t)x;
}

// The lowest optimal configuration of one entry of a vertex described by class
// fill terms, by one wave: w[k] = the configurations of its layout digits (z
// first when it has one).
template <typename KeyT>
__device__ __forceinline__ uint32_t lazy_argmin(const ClassArgs &a, const uint32_t (&w)[kMaxDep]) {
    using Ops = KeyOps<KeyT>;
    using Val = typename Ops::Val;
    constexpr int U = 4;   // configurations in flight per lane
    const uint32_t lane = threadIdx.x & 63, z = a.has_z ? 1 : 0, K = a.K;
    KeyT best = Ops::sentinel();
    for (uint32_t c0 = lane; c0 < K; c0 += 64 * U) {
        KeyT x[U];
#pragma unroll
        for (int u = 0; u < U; u++) x[u] = glb<KeyT>(a.Lk)[min(c0 + 64 * u, K - 1)];
        auto edge = [&](const uint64_t *sc, const uint64_t *so, const void *fc, const void *fo, uint32_t o) {
            const uint64_t s = glb<uint64_t>(so)[o];
            const KeyT f = glb<KeyT>(fo)[o];
            uint64_t sg[U];
            KeyT fg[U];
#pragma unroll
            for (int u = 0; u < U; u++) {
                const uint32_t c = min(c0 + 64 * u, K - 1);
                sg[u] = glb<uint64_t>(sc)[c];
                fg[u] = glb<KeyT>(fc)[c];
            }
#pragma unroll
            for (int u = 0; u < U; u++) x[u] = Ops::add(x[u], sg[u] == s ? (KeyT)0 : Ops::min(f, fg[u]));
        };
        if (z) edge(a.sig_zc, a.sig_zo, a.fzc, a.fzo, w[0]);
        for (uint32_t t = 0; t < a.ne; t++) {
            uint32_t o = 0;
            for (int k = 0; k < kMaxDep; k++) o = k == (int)(z + a.e[t].dig) ? w[k] : o;
            edge(a.e[t].sig_c, a.e[t].sig_o, a.e[t].f_c, a.e[t].f_o, o);
        }
        for (uint32_t t = 0; t < a.nt; t++) {
            uint64_t o = 0;
            for (int k = 0; k < kMaxDep; k++)
                if (k >= (int)z && k - (int)z < (int)a.nR) o += (uint64_t)w[k] * a.t[t].sd[k - z];
            KeyT tv[U];
#pragma unroll
            for (int u = 0; u < U; u++)
                tv[u] = __builtin_bit_cast(KeyT, glb<Val>(a.t[t].ptr)[o + (uint64_t)min(c0 + 64 * u, K - 1) * a.t[t].sc]);
#pragma unroll
            for (int u = 0; u < U; u++) x[u] = Ops::add(x[u], tv[u]);
        }
#pragma unroll
        for (int u = 0; u < U; u++) best = Ops::min(best, x[u]);
    }
    for (uint32_t m = 32; m > 0; m >>= 1) best = Ops::min(best, shfl_xor_key(best, (int)m));
    Val v;
    uint32_t cc;
    Ops::split(best, a.bits, 0, v, cc);
    return cc;
}

}  // namespace pase
