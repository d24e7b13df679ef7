// Host side of libpase: graph validation, configuration enumeration, the
// GenerateSeq vertex order (Fig. 3), connected sets / dependent sets /
// connected subsets (Sec. III-B), per-vertex DP plans and the device memory
// layout.  No HIP calls here: everything is pure host computation so it can be
// exercised without a GPU.
#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstring>
#include <numeric>
#include <unordered_map>

#include "internal.h"

using namespace pase;

namespace pase {

pase_status fail(pase_graph_t g, pase_status st, const std::string &msg) {
    if (g) g->err = msg;
    return st;
}

static bool mul_ok(uint64_t a, uint64_t b, uint64_t *out) { return !__builtin_mul_overflow(a, b, out); }
static bool add_ok(uint64_t a, uint64_t b, uint64_t *out) { return !__builtin_add_overflow(a, b, out); }
static uint64_t align_up(uint64_t x, uint64_t a) { return (x + a - 1) / a * a; }
static uint32_t bits_for(uint32_t K) {
    uint32_t b = 0;
    while ((1u << b) < K) b++;
    return b;
}

// Upper bounds of the DP quantities at every sequence position i, used to
// size the keys.  Q_i(phi, c) -- the layer cost of v_i at c, plus r * t_x of
// every edge joining v_i and a later vertex, plus the table lookup of every
// connected subset -- is at most maxL(v_i) + sum maxR + sum Tmax_j.  The table
// entry T_i(phi) = min_c Q_i(phi, c) is at most Q_i(phi, c0) for any single c0:
// with model costs c0 is the cheapest of the unsplit configuration (cost F)
// and the ones that split a single dim p ways (costs evaluated exactly); with
// caller-given costs it is the cheapest layer configuration.  These bounds
// follow the recurrence instead of summing every cost of the graph, so deep
// graphs keep exact fp64 keys.  They depend on the sequence and the costs, not
// on the fills, and are evaluated once for these (plan.qmax, plan.tmax).
// false: a bound exceeds 64 bits.
static bool eval_bounds(pase_graph_t g) {
    Plan &P = g->plan;
    const size_t n = P.v.size();
    P.qmax.assign(n, 0);
    P.tmax.assign(n, 0);
    for (size_t i = 0; i < n; i++) {
        const VPlan &vp = P.v[i];
        const int v = vp.vi;
        uint64_t hi = g->maxL[v], lo;
        if (g->overridden) {
            hi = 0;
            lo = ~0ull;
            for (uint32_t c = 0; c < g->K[v]; c++) {
                hi = std::max(hi, g->ov_layer[g->ov_layer_off[v] + c]);
                lo = std::min(lo, g->ov_layer[g->ov_layer_off[v] + c]);
            }
        } else {
            // the exact cost of single configurations: unsplit (F: no partial
            // sums, no replicas), and each dim k split p ways; every term of
            // these is bounded by the parts of maxL, so nothing overflows
            const pase_vertex_desc &d = g->V[v];
            const uint64_t F = g->flops[v], W = g->weight_n[v], p = g->p;
            lo = F;
            for (uint32_t k = 0; k < d.ndims; k++) {
                uint64_t c = (F + p - 1) / p;
                if ((d.reduce_mask >> k) & 1u) c += g->r * (p - 1) * g->keep_n[v];
                if (W && !((d.weight_mask >> k) & 1u)) c += g->r * (2 * W - 2 * W / p);
                // the halo of the split dim itself: the other input dims are unsplit
                if (g->halo && d.halo[k]) c += g->r * 2 * (uint64_t)d.halo[k] * g->halo_n[v][k];
                lo = std::min(lo, c);
            }
        }
        uint64_t rest = 0;
        for (int e : vp.edges) {
            uint64_t m = g->maxR[e];
            if (g->overridden) {
                m = 0;
                const uint64_t cnt = (uint64_t)g->K[g->E[e].src] * g->K[g->E[e].dst];
                for (uint64_t k = 0; k < cnt; k++) m = std::max(m, g->ov_edge[g->ov_edge_off[e] + k]);
            }
            if (!add_ok(rest, m, &rest)) return false;
        }
        for (const TermRef &t : vp.terms)
            if (!add_ok(rest, P.tmax[t.j], &rest)) return false;
        if (!add_ok(hi, rest, &P.qmax[i]) || !add_ok(lo, rest, &P.tmax[i])) return false;
    }
    return true;
}

bool cost_bounds(pase_graph_t g) {
    if (g->plan.bounds < 0) g->plan.bounds = eval_bounds(g) ? 1 : 0;
    return g->plan.bounds == 1;
}

// Key type: fp64 when every key (cost * 2^bits + c) of every position stays
// within 2^53 so that double arithmetic on them is exact integer arithmetic;
// otherwise uint64 when it stays within 2^64; otherwise 128-bit keys, which
// hold cost * 2^bits + c exactly as long as every cost sum fits 64 bits (the
// costs and tables the C ABI reports are uint64); when a cost bound itself
// passes 64 bits, overflow.  A stored table entry T_j (in its reader's key
// space) is at most the reader's bound.  key_mode 1 / 2 force uint64 (when
// the keys fit) / 128-bit keys.
uint32_t choose_key_type(pase_graph_t g, pase_status *st) {
    *st = PASE_OK;
    if (!cost_bounds(g)) { *st = PASE_ERR_OVERFLOW; return 0; }
    const std::vector<uint64_t> &qmax = g->plan.qmax;
    unsigned __int128 top = 0;
    for (size_t i = 0; i < qmax.size(); i++) {
        // largest key: qmax * 2^bits + (2^bits - 1) < (qmax + 1) * 2^bits
        const unsigned __int128 t = ((unsigned __int128)qmax[i] + 1) << g->plan.v[i].bits;
        top = std::max(top, t);
    }
    if (g->key_mode == 2) return 2;
    if (g->key_mode == 0 && top <= ((unsigned __int128)1 << 53)) return 0;
    if (top <= ((unsigned __int128)1 << 64)) return 1;
    return 2;
}

uint32_t key_bytes(pase_graph_t g) { return g->plan_wide ? 16u : 8u; }

}  // namespace pase

// ------------------------------------------------------------------ create / destroy
extern "C" pase_status pase_graph_create(const pase_vertex_desc *v, uint32_t nv,
                                         const pase_edge_desc *e, uint32_t ne,
                                         const pase_cost_params *params, pase_graph_t *out) {
    if (!v || !out || nv == 0 || (ne > 0 && !e)) return PASE_ERR_INVALID_ARGUMENT;
    if (nv > (1u << 20) || ne > (1u << 24)) return PASE_ERR_INVALID_ARGUMENT;
    for (uint32_t i = 0; i < nv; i++) {
        if (v[i].ndims < 1 || v[i].ndims > kMaxDims) return PASE_ERR_INVALID_ARGUMENT;
        for (uint32_t k = 0; k < v[i].ndims; k++)
            if (v[i].size[k] == 0) return PASE_ERR_INVALID_ARGUMENT;
        if (v[i].reduce_mask >> v[i].ndims) return PASE_ERR_INVALID_ARGUMENT;
        if (v[i].weight_mask >> v[i].ndims) return PASE_ERR_INVALID_ARGUMENT;
        if (v[i].input_mask >> v[i].ndims) return PASE_ERR_INVALID_ARGUMENT;
        for (uint32_t k = 0; k < kMaxDims; k++)
            if (v[i].halo[k] && (k >= v[i].ndims || !((v[i].input_mask >> k) & 1u) || v[i].halo[k] > (1u << 16)))
                return PASE_ERR_INVALID_ARGUMENT;
    }
    for (uint32_t k = 0; k < ne; k++) {
        const pase_edge_desc &d = e[k];
        if (d.src >= nv || d.dst >= nv || d.src == d.dst) return PASE_ERR_INVALID_ARGUMENT;
        if (d.rank > kMaxDims || d.elems == 0) return PASE_ERR_INVALID_ARGUMENT;
        for (uint32_t t = 0; t < d.rank; t++) {
            if (d.src_dim[t] < -1 || d.src_dim[t] >= (int32_t)v[d.src].ndims)
                return PASE_ERR_INVALID_ARGUMENT;
            if (d.dst_dim[t] < -1 || d.dst_dim[t] >= (int32_t)v[d.dst].ndims)
                return PASE_ERR_INVALID_ARGUMENT;
        }
    }
    auto *g = new pase_graph_s();
    g->V.assign(v, v + nv);
    if (ne) g->E.assign(e, e + ne);
    if (params) {
        g->r = params->comm_weight ? params->comm_weight : 8;
        if (params->seq_rule > 1) { delete g; return PASE_ERR_INVALID_ARGUMENT; }
        g->seq_rule = params->seq_rule;
    }
    g->nbr.assign(nv, {});
    for (const auto &d : g->E) {
        g->nbr[d.src].push_back((int)d.dst);
        g->nbr[d.dst].push_back((int)d.src);
    }
    for (auto &l : g->nbr) {
        std::sort(l.begin(), l.end());
        l.erase(std::unique(l.begin(), l.end()), l.end());
    }
    // weak connectivity (computation graphs are weakly connected, Sec. II)
    std::vector<char> seen(nv, 0);
    std::vector<int> stack{0};
    seen[0] = 1;
    size_t count = 1;
    while (!stack.empty()) {
        int x = stack.back();
        stack.pop_back();
        for (int y : g->nbr[x])
            if (!seen[y]) { seen[y] = 1; count++; stack.push_back(y); }
    }
    if (count != nv) { delete g; return PASE_ERR_NOT_CONNECTED; }
    *out = g;
    return PASE_OK;
}

extern "C" void pase_graph_destroy(pase_graph_t g) {
    if (!g) return;
    device_release(g);
    delete g;
}

extern "C" const char *pase_last_error(pase_graph_t g) { return g ? g->err.c_str() : ""; }

// ------------------------------------------------------------------ planning
namespace {

// Breadth-first traversal from vertex 0, neighbours in ascending id order:
// the sequence of the breadth-first recurrence (eq. 2).
std::vector<int> bfs_order(pase_graph_t g) {
    const size_t n = g->V.size();
    std::vector<int> order;
    order.reserve(n);
    std::vector<char> seen(n, 0);
    order.push_back(0);
    seen[0] = 1;
    for (size_t h = 0; h < order.size(); h++)
        for (int u : g->nbr[order[h]])      // ascending, deduplicated
            if (!seen[u]) { seen[u] = 1; order.push_back(u); }
    return order;
}

// GenerateSeq (Fig. 3): repeatedly sequence the unsequenced vertex with the
// smallest d-set (ties: lowest vertex id); every member of its d-set absorbs
// it.  rule 0 keeps a vertex out of its own d-set; rule 1 applies the printed
// update literally.  The d-set at selection (minus the vertex) is D(i)
// (Theorem 2).  Bitsets, one per vertex.  With a fixed `order` the same
// absorption runs along that order instead of the smallest-d-set choice: the
// d-set of a vertex then still holds the unsequenced neighbours of the
// sequenced component it would join, so at selection it is D(i) =
// N(X(i)) after i for that order (for a breadth-first order, D_B(i)).
void generate_seq(pase_graph_t g, std::vector<int> &seq, std::vector<std::vector<int>> &Dpos,
                  const std::vector<int> *order = nullptr) {
    const size_t n = g->V.size(), W = (n + 63) / 64;
    std::vector<uint64_t> d(n * W, 0);
    for (size_t v = 0; v < n; v++)
        for (int u : g->nbr[v]) d[v * W + u / 64] |= 1ull << (u % 64);
    // |u.d| is kept per vertex, counting the members that come and go
    auto count = [&](size_t u) {
        int sz = 0;
        for (size_t w = 0; w < W; w++) sz += __builtin_popcountll(d[u * W + w]);
        return sz;
    };
    std::vector<int> size(n);
    for (size_t u = 0; u < n; u++) size[u] = count(u);
    // vertices not sequenced yet, in no particular order: the pick is the
    // smallest (|u.d|, vertex id), so the scan order does not matter
    std::vector<int> left(n), where(n);
    std::iota(left.begin(), left.end(), 0);
    std::iota(where.begin(), where.end(), 0);
    seq.clear();
    Dpos.assign(n, {});
    for (size_t i = 0; i < n; i++) {
        size_t best = n;
        if (order) {
            best = (size_t)(*order)[i];
        } else {
            for (int u : left)
                if (best == n || size[u] < size[best] || (size[u] == size[best] && (size_t)u < best)) best = (size_t)u;
        }
        const size_t vi = best;
        // remove vi from the unsequenced set (swap with the last)
        const int at = where[vi], tail = left.back();
        left[at] = tail;
        where[tail] = at;
        left.pop_back();
        seq.push_back((int)vi);
        // D(i) = vi.d (ascending vertex id): the set bits of its row
        for (size_t w = 0; w < W; w++)
            for (uint64_t bits = d[vi * W + w]; bits; bits &= bits - 1) {
                const size_t u = w * 64 + (size_t)__builtin_ctzll(bits);
                if (u != vi) Dpos[i].push_back((int)u);
            }
        for (int v : Dpos[i]) {
            uint64_t *dv = &d[(size_t)v * W];
            for (size_t w = 0; w < W; w++) {
                uint64_t more = d[vi * W + w] & ~dv[w];
                if (g->seq_rule == 0 && w == (size_t)v / 64) more &= ~(1ull << (v % 64));
                dv[w] |= more;
                for (; more; more &= more - 1) size[v]++;
            }
            const uint64_t out = 1ull << (vi % 64);
            size[v] -= (dv[vi / 64] & out) != 0;
            dv[vi / 64] &= ~out;
        }
    }
}

// column chunk widths of the row kernel (keys per lane and c, read as one
// scalar round trip of up to two s_load_dwordx16 plus a smaller load)
const uint32_t kTZ[] = {8, 12, 14, 16, 24, 28};

struct RowsChoice {
    bool ok = false;
    double cost = 0;
    int z = -1;
    std::vector<int> O, R;
    uint32_t TZ = 0, TM = 1, na = 0, parts = 1, nsplit = 1;
    uint64_t MO = 1, MR = 1;
};

// Estimated fill time (us) of one row-kernel vertex for a tile shape, with the
// best number of c parts per tile (waves of a workgroup) and c splits (across
// workgroups) -- or the forced ones.  The time is the larger of the throughput
// bound (the busiest SIMD's waves, each issuing a VALU op every 4 cycles) and
// the latency bound of a single wave: per value of c at least one memory round
// trip for the operands prefetched one c ahead (~450 cycles; column-less tiles
// keep 8 values of c in flight, ~360 cycles per c), or its own VALU work at
// about one op per 8 cycles.  Column-less tiles also stream their large
// lookups (stream_bytes: the multi-digit tables they read, each entry once;
// the one-digit row blocks stay in cache) at ~3.3 TB/s; when that stream binds,
// the estimates of several part counts tie, and the most parts win: more
// waves keep more loads in flight (measured on the Transformer's streaming
// fills: 287 us with one part, 244 us with two or four).  A c split adds a
// reduction launch (~10 us with its gap) and the partial keys' traffic; the
// column block is built at ~115 G elements/s.
struct TileTime {
    double us;
    uint32_t parts, nsplit;
};

TileTime tile_time(uint64_t MO, uint64_t MR, uint32_t Kz, uint32_t K, uint32_t na, uint32_t tz, uint32_t tm,
                   uint32_t force_parts, uint32_t force_splits, double stream_bytes) {
    const double clk = 2400.0;   // cycles per us
    const uint64_t nch = (Kz + tz - 1) / tz;
    const uint64_t tiles = MO * ((MR + 64 * tm - 1) / (64 * tm)) * nch;
    const uint64_t N = MO * MR * (uint64_t)Kz;
    const double prep_us = (double)MO * K * nch * tz / 1.15e5;
    TileTime best{1e300, 1, 1};
    for (uint32_t P = 1; P <= 4; P *= 2) {
        if (force_parts && P != force_parts) continue;
        for (uint32_t S = 1; S <= 64; S *= 2) {
            if (force_splits && S != 1) break;
            const uint32_t Sx = force_splits ? std::min(force_splits, K) : S;
            if (!force_splits && S > 1 && K < 8 * P * S) break;
            const double cw = std::ceil(std::ceil((double)K / Sx) / P);
            double wave_cyc, lat_cyc, bw_us = 0;
            if (tz >= 8) {
                // VALU slots per c: two per cell, the row-term adds, and (measured)
                // a few for wide chunks (> 16 keys: no scalar-load overlap) and
                // for two rows per lane (more VGPRs, fewer waves).  Every row-term
                // load is a wave-wide vector load that keeps the CU's texture
                // address unit ~16 cycles busy; shared by four SIMDs, that costs
                // ~15 VALU slots per load per wave when all SIMDs are busy; the
                // two overlap imperfectly (fitted: the smaller adds a quarter).
                const double valu = 2.0 * tz * tm + tm * (na > 0 ? na - 1.0 : 0.0) + 1.0 + (tz > 16 ? 2.0 : 0.0) +
                                    (tm == 2 ? 2.0 : 0.0);
                const double ta = 14.7 * na * tm;
                double per_c = std::max(valu, ta) + 0.25 * std::min(valu, ta);
                // a column block larger than the L2s is read from HBM: a scalar
                // round trip then takes ~2000 cycles, ~60 slots per wave with
                // eight waves per SIMD -- hidden behind one c of work when the
                // loads of c + 1 are in flight (up to 16 keys), exposed when not
                if ((double)MO * K * nch * tz * 8 > 16e6) per_c = tz > 16 ? per_c + 62.0 : std::max(per_c, 62.0);
                const double tail = tz * tm * (P > 1 ? 8.0 : 6.0);
                wave_cyc = 4.0 * (cw * per_c + tail);
                lat_cyc = cw * std::max(8.0 * per_c, 450.0) + 8.0 * tail;
            } else {
                wave_cyc = 4.0 * cw * (2.0 * tm + tm * (na > 0 ? na - 1.0 : 0.0) + 1.0);
                lat_cyc = 360.0 * cw;
                bw_us = stream_bytes / 3.3e6;
            }
            // the busiest SIMD: the average share plus, on average, half a wave
            const double W = (double)tiles * P * Sx;
            const double t_tp = (W / 1024.0 + 0.5) * wave_cyc / clk;
            double us = std::max(std::max(t_tp, lat_cyc / clk), bw_us) + prep_us;
            if (Sx > 1) us += 10.0 + (double)N * Sx * 16 / 5e6;
            // parts ascend: a column-less tie goes to the later, larger count
            const bool tie_more_parts = tz < 8 && Sx == 1 && best.nsplit == 1 && us <= best.us * (1.0 + 1e-9);
            if (us < best.us || tie_more_parts) best = {us, P, Sx};
        }
    }
    return best;
}

// The best tile shape of one column choice (tz, tm: forced columns and rows per
// lane, 0 = free).  Vertices of one graph often share a shape (the layers of a
// stack): the tile model is evaluated once per distinct argument tuple.
struct TileChoice {
    bool ok = false;
    uint32_t TZ = 0, TM = 1;
    TileTime t{0, 1, 1};
};

TileChoice tile_choice(uint64_t MO, uint64_t MR, int z, uint32_t Kz, uint32_t K, uint32_t na, uint32_t force_tz,
                       uint32_t force_tm, uint32_t force_parts, uint32_t force_splits, double stream_bytes) {
    struct Key {
        uint64_t MO, MR;
        uint32_t Kz, K, na, tz, tm, parts, splits, col;
        double sb;
        bool operator==(const Key &o) const {
            return MO == o.MO && MR == o.MR && Kz == o.Kz && K == o.K && na == o.na && tz == o.tz && tm == o.tm &&
                   parts == o.parts && splits == o.splits && col == o.col && sb == o.sb;
        }
    };
    struct Hash {
        size_t operator()(const Key &k) const {
            uint64_t h = k.MO * 0x9E3779B97F4A7C15ull ^ (k.MR + 0x632BE59BD9B4E019ull) ^ (uint64_t)k.sb;
            for (uint32_t x : {k.Kz, k.K, k.na, k.tz, k.tm, k.parts, k.splits, k.col}) h = (h ^ x) * 0x100000001B3ull;
            return (size_t)h;
        }
    };
    thread_local std::unordered_map<Key, TileChoice, Hash> memo;
    const Key key{MO, MR, Kz, K, na, force_tz, force_tm, force_parts, force_splits, z >= 0 ? 1u : 0u, stream_bytes};
    auto it = memo.find(key);
    if (it != memo.end()) return it->second;
    if (memo.size() > 8192) memo.clear();
    TileChoice c;
    auto consider = [&](uint32_t tz) {
        const uint64_t nch = (Kz + tz - 1) / tz;
        if (MO * K * nch * tz > kMaxTableEntries) return;
        for (uint32_t tm = 1; tm <= 2; tm++) {
            if (force_tm && tm != force_tm) continue;
            // more than 32 accumulators per lane cost waves (VGPRs)
            if (!force_tm && !force_tz && tz * tm > 32) continue;
            const TileTime t = tile_time(MO, MR, Kz, K, na, tz, tm, force_parts, force_splits, stream_bytes);
            if (!c.ok || t.us < c.t.us) c = {true, tz, tm, t};
        }
    };
    if (z < 0) consider(1);
    else
        for (uint32_t tz : kTZ)
            if (!force_tz || tz == force_tz) consider(tz);
    memo.emplace(key, c);
    return c;
}

}  // namespace

// Fused minima.  A row-kernel vertex i2 without a column digit whose only
// lookup is the table of i1 -- a row-kernel vertex whose column digit is v_i2,
// with no outer digits, the same row digits and neither of them split over c
// -- streams all of T_i1 once to take, per row, a minimum over c = z.  i1's fill
// forms those keys itself in its epilogue instead (T_i1 has no other reader),
// so T_i1 is neither written to nor read back from HBM, and i2 keeps a
// one-split reduction of the combined keys.  i2's prep blocks hold static
// costs only (its one lookup is read in the kernel), so they are built in
// i1's prep launch, before i1's fill.  Both run on one lane.
static void fuse_minima(pase_graph_t g, Plan &P) {
    (void)g;
    const int n = (int)P.v.size();
    for (int i2 = 0; i2 < n; i2++) {
        VPlan &b = P.v[i2];
        if (b.kernel != kRows || b.classes || b.joint >= 0 || b.z >= 0 || b.nsplit != 1 || b.terms.size() != 1 || b.terms[0].dig.size() < 2)
            continue;
        const int i1 = b.terms[0].j;
        VPlan &a = P.v[i1];
        if (a.kernel != kRows || a.classes || a.joint >= 0 || a.z != b.vi || !a.O.empty() || a.R != b.R || a.nsplit != 1 || a.consumer != i2 ||
            a.lane != b.lane || a.fuse_into >= 0 || a.fused_from >= 0)
            continue;
        a.fuse_into = i2;
        b.fused_from = i1;
        P.fused++;
    }
}

// Hoisted preps (level layout: one stream, slots = levels).  A vertex's prep builds its key-space blocks
// from static costs and from the tables of the lookups that enter blocks (the
// column block's and the one-digit row blocks'; multi-digit lookups on row
// digits are read by the fill itself).  When the last of those tables is
// filled two or more slots before the vertex's own, and the blocks are large
// (PASE_OPT_HOIST_ELEMS, by default 2^20 elements: ~10 us or more of HBM
// writes), the prep runs on a side stream instead of in the vertex's slot,
// started right after that slot, on a grid of one workgroup per CU: it then
// takes several times longer but leaves most of the GPU to the launches of
// the slots in between (a full-size prep grid beside them slows them down
// more than it saves).
//
// A joint fill has a half fill in place of a prep: it runs in the slot of the
// vertex whose side it computes, and counts as hoisted (prep_after is that
// slot) when it reads tables and that slot is two or more before the fill's.
static void hoist_preps(pase_graph_t g, Plan &P, bool lanes) {
    for (auto &vp : P.v) {
        if (vp.joint >= 0) {
            const VPlan &vj = P.v[vp.joint];
            if (!vp.jearly || vj.terms.empty() || vj.slot + 2 > vp.slot) continue;
            vp.prep_after = vj.slot;
            vp.prep_lane = vj.lane;
            continue;
        }
        if ((vp.kernel != kRows && vp.kernel != kGeneric) || vp.classes || vp.fused_from >= 0 || vp.fuse_into >= 0 ||
            (vp.absorbed >= 0 && P.v[vp.absorbed].exch))
            continue;
        uint64_t elems = 0;
        int ready = -1;
        int lane = -1;            // lane of the tables the blocks read (-2: more than one)
        auto note = [&](int j) {
            ready = std::max(ready, P.v[j].slot);
            lane = lane == -1 || lane == P.v[j].lane ? P.v[j].lane : -2;
        };
        if (vp.kernel == kRows) {
            elems = vp.MO * vp.K * vp.ldz;
            for (int u : vp.R) elems += (uint64_t)vp.K * g->K[u];
            std::vector<int> OZ = vp.O;
            if (vp.z >= 0) OZ.push_back(vp.z);
            for (const auto &t : vp.terms) {
                bool all = true;
                for (int u : t.dig) all &= std::find(OZ.begin(), OZ.end(), u) != OZ.end();
                const bool row1 = t.dig.size() == 1 && std::count(vp.R.begin(), vp.R.end(), t.dig[0]);
                if (all || row1) note(t.j);
            }
        } else {
            elems = vp.K;
            for (int u : vp.D) elems += (uint64_t)vp.K * g->K[u];
            for (const auto &t : vp.terms)
                if (t.dig.size() <= 1) note(t.j);
        }
        // with lanes, the prep runs at the end of the group (slot `ready`, at
        // least 0) of the lane whose tables it reads (the vertex's own when it
        // reads none): stream order puts it after those fills, and the
        // vertex's group waits for that lane up to that slot anyway -- or
        // shares its stream -- so the prep precedes the fill
        if (lanes) {
            if (lane == -2) continue;
            ready = std::max(ready, 0);
        }
        if (g->hoist_elems && elems >= g->hoist_elems && ready + 2 <= vp.slot) {
            vp.prep_after = ready;
            vp.prep_lane = lanes && lane >= 0 ? lane : vp.lane;
            P.hoisted++;
        }
    }
}

// Bulk lane schedule.  Row-kernel vertices planned to take at least bulk_us
// (the large fills, which keep the whole GPU busy on their own) run on lane 1
// (the caller's stream), and so does every vertex that reads a table of lane 1
// (it has to wait for that fill anyway); every other vertex -- one whose
// producers are all small -- runs on lane 0 (a side stream), level by
// level, at the highest wave priority.  A level group of lane 0 then never
// waits for a large fill, so a chain of small dependent vertices runs beside
// the large fills instead of after them.  Producers precede their reader in
// the sequence, so one pass suffices.
// (A class fill counts from a quarter of the threshold: it is bound by the
// stores of its table, which hold up the other lane's loads as well.)
// A vertex without a table of its own is where its half fill's reader is.
static bool bulk_fill(const Plan &P, const VPlan &vp, double bulk_us) {
    return (vp.kernel == kRows && vp.est_us * (vp.classes || vp.joint >= 0 ? 4.0 : 1.0) >= bulk_us) ||
           (vp.absorbed >= 0 && bulk_fill(P, P.v[vp.absorbed], bulk_us));
}

static void assign_bulk_lanes(Plan &P, double bulk_us) {
    for (auto &vp : P.v) {
        bool bulk = bulk_fill(P, vp, bulk_us);
        for_reads(P, vp, [&](int j) { bulk |= P.v[j].lane == 1; });
        vp.lane = bulk ? 1 : 0;
    }
}

// Split chains schedule.  The first kSplitBatchedLevels levels -- the leaves,
// where the largest fills and most small vertices are -- run level by level
// on lane 1, batched as in the level schedule.  After them, a row-kernel
// vertex planned at bulk_us or more, and every vertex reading a table such a
// vertex (or one of its readers) fills after the batched levels, runs on lane
// 1 too; the remaining small vertices run on lane 0.  A lane-0 group waits
// once for the batched levels whose tables it reads and then runs beside lane
// 1, so a chain of small vertices and a chain of larger fills no longer wait
// for each other level by level.
static void assign_split_lanes(Plan &P, double bulk_us) {
    for (auto &vp : P.v) {
        bool one = vp.level < kSplitBatchedLevels || bulk_fill(P, vp, bulk_us);
        for_reads(P, vp, [&](int j) { one |= P.v[j].lane == 1 && P.v[j].level >= kSplitBatchedLevels; });
        vp.lane = one ? 1 : 0;
    }
}

static double ms_since(std::chrono::steady_clock::time_point t0) {
    return std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
}

// What the plan takes from the graph alone: the sequence, the dependent sets,
// lookups, edges and table sizes of every position, and the dependency levels.
static pase_status build_structure(pase_graph_t g) {
    const auto t0 = std::chrono::steady_clock::now();
    const int n = (int)g->V.size();
    Plan &P = g->plan;
    P = Plan();
    std::vector<std::vector<int>> Dpos;
    if (g->order_mode == 1) {
        const std::vector<int> order = bfs_order(g);
        generate_seq(g, P.seq, Dpos, &order);
    } else {
        generate_seq(g, P.seq, Dpos);
    }
    P.pos.assign(n, 0);
    for (int i = 0; i < n; i++) P.pos[P.seq[i]] = i;
    P.v.assign(n, VPlan());

    // edges of each vertex, in edge order
    std::vector<std::vector<int>> incident(n);
    for (size_t k = 0; k < g->E.size(); k++) {
        incident[g->E[k].src].push_back((int)k);
        incident[g->E[k].dst].push_back((int)k);
    }
    // components of the graph induced on positions < i, grown one position at
    // a time (union-find over vertex ids); each set remembers its last position
    std::vector<int> uf(n), last(n, -1), seen(n, -1);
    std::iota(uf.begin(), uf.end(), 0);
    auto find = [&](int x) {
        while (uf[x] != x) x = uf[x] = uf[uf[x]];
        return x;
    };
    for (int i = 0; i < n; i++) {
        VPlan &vp = P.v[i];
        vp.vi = P.seq[i];
        vp.K = g->K[vp.vi];
        vp.bits = bits_for(vp.K);
        vp.D = Dpos[i];
        std::sort(vp.D.begin(), vp.D.end());
        if (vp.D.size() > (size_t)kMaxDep)
            return fail(g, PASE_ERR_TOO_LARGE, "dependent set larger than PASE_MAX_DEP");
        P.max_dep = std::max<uint32_t>(P.max_dep, (uint32_t)vp.D.size());
        vp.N = 1;
        for (int w : vp.D)
            if (!mul_ok(vp.N, g->K[w], &vp.N) || vp.N > kMaxTableEntries)
                return fail(g, PASE_ERR_TOO_LARGE, "a DP table exceeds 2^31 entries");
        // S(i): the components of V<i that v_i touches, each represented by its
        // last position j (X(i) - {v_i} is their union)
        for (int s : g->nbr[vp.vi]) {
            if (P.pos[s] >= i) continue;
            const int rt = find(s);
            if (seen[rt] == i) continue;
            seen[rt] = i;
            const int jmax = last[rt];
            TermRef t;
            t.j = jmax;
            bool has_vi = false;
            for (int u : P.v[jmax].D) {
                if (u == vp.vi) { has_vi = true; continue; }
                if (!std::binary_search(vp.D.begin(), vp.D.end(), u))
                    return fail(g, PASE_ERR_INTERNAL, "D(j) not within D(i) + v_i");
                t.dig.push_back(u);
            }
            if (!has_vi) return fail(g, PASE_ERR_INTERNAL, "v_i missing from D(j)");
            if (P.v[jmax].consumer != -1) return fail(g, PASE_ERR_INTERNAL, "table read twice");
            P.v[jmax].consumer = i;
            vp.terms.push_back(t);
        }
        // v_i joins the components it touches and is their last position
        last[vp.vi] = i;
        for (int s : g->nbr[vp.vi])
            if (P.pos[s] < i) {
                const int a = find(s), b = find(vp.vi);
                if (a != b) uf[a] = b;
            }
        last[find(vp.vi)] = i;
        for (int k : incident[vp.vi]) {
            const auto &d = g->E[k];
            const int other = (int)d.src == vp.vi ? (int)d.dst : (int)d.src;
            if (P.pos[other] > i) vp.edges.push_back(k);
        }
        P.cells += vp.N * vp.K;
        P.entries += vp.N;
    }
    for (int i = 0; i + 1 < n; i++) {
        if (P.v[i].consumer < 0) return fail(g, PASE_ERR_INTERNAL, "table never read");
        P.v[i].out_shift = P.v[P.v[i].consumer].bits;
    }
    // dependency level: vertices of one level read no table of each other
    for (int i = 0; i < n; i++) {
        P.v[i].level = 0;
        for (const auto &t : P.v[i].terms) P.v[i].level = std::max(P.v[i].level, P.v[t.j].level + 1);
    }
    g->stats.seq_ms = ms_since(t0);
    return PASE_OK;
}

// The plan's structure alone, for other fills of the same graph.
static void reset_fills(Plan &P) {
    Plan q;
    q.seq.swap(P.seq);
    q.pos.swap(P.pos);
    q.cells = P.cells;
    q.entries = P.entries;
    q.max_dep = P.max_dep;
    q.bounds = P.bounds;
    q.qmax.swap(P.qmax);
    q.tmax.swap(P.tmax);
    q.v.resize(P.v.size());
    for (size_t i = 0; i < P.v.size(); i++) {
        VPlan &a = q.v[i], &b = P.v[i];
        a.vi = b.vi;
        a.K = b.K;
        a.bits = b.bits;
        a.D.swap(b.D);
        a.N = b.N;
        a.edges.swap(b.edges);
        a.terms.swap(b.terms);
        a.consumer = b.consumer;
        a.out_shift = b.out_shift;
        a.level = b.level;
    }
    P = std::move(q);
}

// The fill, layout and lane of every position.
static pase_status plan_fills(pase_graph_t g) {
    const auto t1 = std::chrono::steady_clock::now();
    Plan &P = g->plan;
    const int n = (int)P.v.size();
    // ---- kernel choice and T_i layout
    // threads of the generic and direct fills walk the table in layout order:
    // follow the memory order of the largest lookup that spans several digits
    // so that its reads coalesce
    auto gather_layout = [&](const VPlan &vp) {
        int big = -1;
        for (size_t t = 0; t < vp.terms.size(); t++)
            if (vp.terms[t].dig.size() >= 2 && (big < 0 || P.v[vp.terms[t].j].N > P.v[vp.terms[big].j].N))
                big = (int)t;
        if (big < 0) return vp.D;
        const VPlan &pj = P.v[vp.terms[big].j];
        std::vector<int> order;
        for (int u : pj.layout)
            if (u != vp.vi) order.push_back(u);   // slowest first in T_j
        for (int u : vp.D)
            if (std::find(order.begin(), order.end(), u) == order.end()) order.insert(order.begin(), u);
        return order;
    };
    // the direct fill pays where it removes launches: for a whole level (the
    // vertices of one launch group), or any vertex when each has its own slot
    int maxlev = 0;
    for (int i = 0; i < n; i++) maxlev = std::max(maxlev, P.v[i].level);
    std::vector<char> level_small((size_t)maxlev + 1, 1);
    for (int i = 0; i < n; i++)
        if (P.v[i].N * P.v[i].K > g->direct_cells) level_small[P.v[i].level] = 0;
    // plan_one(i, ftz, ftm, no_split): kernel, tile and layout of position i;
    // ftz/ftm (0 = free) force the row kernel's columns and rows per lane for
    // this vertex and rule out the column-less form; no_split rules out a c
    // split
    // 128-bit keys: every vertex on prep + the generic kernel
    const int kernel_mode = g->plan_wide ? 1 : g->kernel_mode;
    // Class fill: with the split match model and no tile knob set, a digit z
    // that meets v_i in one edge and in no lookup.  The digit with the most
    // configurations leaves the fewest rows.  K * rest instead of K * rest * Kz
    // cells and no prep launch (2.05 -> 0.24 ms on the Transformer's largest
    // level at p = 64, 17 -> 6 us on its small chain vertices), at more work
    // per cell: not where that digit is small (dense_faster below).  A direct
    // vertex without such a digit takes the same kernel's plain minimum (8.2 -> 5.5 us per launch on
    // the residual CNN at p = 8).  The tile knobs and a hoisting threshold
    // below its default (0, no hoisting, is none) ask for the dense fills and
    // their preps, which they then get.  With the volume model a direct vertex
    // takes the plain minimum as well, each edge's matrix read as a lookup.
    const bool min_ok = kernel_mode == 0 && !g->dense_only && !g->overridden && !g->tile_cols && !g->tile_rows &&
                        !g->tile_parts && !g->c_splits && (!g->hoist_elems || g->hoist_elems >= kHoistElems);
    const bool class_ok = min_ok && !g->volume;
    auto plan_class = [&](int i, bool direct) {
        VPlan &vp = P.v[i];
        const size_t lookups = vp.terms.size() + (g->volume ? vp.edges.size() : 0);
        if (!min_ok || (g->volume && !direct) || vp.K > kClassMaxK || lookups > (size_t)kMaxClassTerms) return false;
        auto edges_to = [&](int w) {
            int k = 0;
            for (int e : vp.edges) k += (int)g->E[e].src == w || (int)g->E[e].dst == w;
            return k;
        };
        int z = -1;
        for (int w : vp.D) {
            bool looked = g->K[w] > kClassMaxK || edges_to(w) != 1;
            for (const auto &t : vp.terms) looked |= std::count(t.dig.begin(), t.dig.end(), w) > 0;
            if (class_ok && !looked && (z < 0 || g->K[w] > g->K[z])) z = w;
        }
        const size_t edges = (g->volume ? 0 : vp.edges.size()) - (z >= 0);
        if ((z < 0 && !direct) || edges > (size_t)kMaxClassEdges) return false;
        const uint64_t rows = vp.N / (z >= 0 ? g->K[z] : 1);
        const uint32_t Kz = z >= 0 ? g->K[z] : 1;
        const uint32_t ne = (uint32_t)edges, nt = (uint32_t)lookups;
        auto fits = [&](uint32_t lr, bool keep) {
            return class_lds(vp.K, Kz, ne, nt, lr, z >= 0, keep, 512) <= kClassMaxLds;
        };
        // rows per workgroup.  Few rows: so many that there is about one
        // workgroup per CU and every lane group has a configuration (X in
        // LDS).  Many rows: 64, a whole wave's, so that the table is stored in
        // full lines; X then fits up to K of about 100, else it is formed
        // twice -- unless that would read a large lookup twice, where fewer
        // rows with X in LDS are better.
        uint64_t looked = 0;
        for (const auto &t : vp.terms) looked += P.v[t.j].N * 8;
        uint32_t lr = 0, threads = 256;
        bool keep = z >= 0;
        const uint32_t most = std::max(vp.K, Kz);
        while (lr < 6 && ((rows >> lr) > 256 || (threads >> lr) > 2 * most) && fits(lr + 1, keep)) lr++;
        if (z >= 0 && lr < 6 && (rows >> 6) > 256 && fits(6, false) && (looked <= (32ull << 20) || lr < kClassStagedRows)) {
            lr = 6;
            keep = false;
        }
        if (!fits(lr, keep)) return false;
        if (lr == 6 && (rows >> 6) > 256) threads = 512;
        vp.keep = keep;
        vp.threads = threads;
        vp.classes = true;
        vp.lr = lr;
        vp.z = z;
        vp.O.clear();
        vp.layout = gather_layout(vp);   // (z first: its entries are rows apart)
        if (z >= 0) {
            vp.layout.erase(std::find(vp.layout.begin(), vp.layout.end(), z));
            vp.layout.insert(vp.layout.begin(), z);
        }
        vp.R.assign(vp.layout.begin() + (z >= 0), vp.layout.end());
        vp.MO = 1;
        vp.MR = rows;
        vp.TZ = 0;
        vp.TM = 1u << lr;
        vp.nsplit = 1;
        vp.cper = vp.K;
        vp.parts = 0;
        vp.stride.assign(vp.layout.size(), 1);
        for (int k = (int)vp.layout.size() - 2; k >= 0; k--) vp.stride[k] = vp.stride[k + 1] * g->K[vp.layout[k + 1]];
        // the table's stores, or the X evaluations
        vp.est_us = 5.0 + std::max((double)vp.N * 10 / 3.5e6,
                                   (double)rows * vp.K * (4.0 + 6.0 * (double)(vp.edges.size() + vp.terms.size())) / 1e7);
        return true;
    };
    // Whether the dense fill of a vertex just planned as a class fill takes less
    // time.  Both sides are fits to 548 measured vertices (K 7 to 924, Kz 5 to
    // 84, up to 2e5 rows, four edges, a lookup or not): the class fill is its
    // launch, the evaluations of X (twice without X in LDS; unstaged, every
    // configuration's data comes from global memory per row), the stores and,
    // staged, a part per row; the dense one its launch and its prep's, the
    // cells, the row terms and the stores.  At K = 924 and 2e5 rows the class fill takes 519 us and the dense one 115 at
    // Kz = 7, 494 and 986 at Kz = 84.  A table that is read whole by a vertex
    // without a column is read more slowly from the class layout, or not formed
    // at all by the dense one (fused minimum): 2.7 us per 1e6 entries.  A vertex
    // that its reader may take into a joint fill stays a class fill.
    auto dense_faster = [&](int i) {
        const VPlan &vp = P.v[i];
        if (vp.z < 0 || vp.consumer < 0) return false;
        const VPlan &b = P.v[vp.consumer];
        uint32_t to_reader = 0;
        for (int e : vp.edges) to_reader += (int)g->E[e].src == b.vi || (int)g->E[e].dst == b.vi;
        bool joinable = to_reader == 1 && b.K >= 24 && g->K[vp.z] >= 24;
        for (const auto &t : vp.terms) joinable &= !std::count(t.dig.begin(), t.dig.end(), b.vi);
        if (joinable) return false;
        bool whole = b.N * b.K > g->direct_cells;
        for (int w : b.D) {
            bool in = false;
            for (const auto &t : b.terms) in |= t.dig.size() >= 2 && std::count(t.dig.begin(), t.dig.end(), w) > 0;
            whole &= in;
        }
        const double cells = 1e-6 * (double)vp.N * vp.K, entries = 1e-6 * (double)vp.N, rows = 1e-6 * (double)vp.MR;
        const double ne = (double)vp.edges.size() - 1, nt = (double)vp.terms.size(), evals = rows * vp.K * (vp.keep ? 1 : 2);
        const double cls = vp.lr >= kClassStagedRows ? 9.0 + 60 * rows + evals * (0.05 + 0.36 * ne + 0.6 * nt) + 1.75 * entries
                                                     : 7.5 + evals * (4.5 + 0.18 * ne + 0.25 * nt) + 1.9 * entries;
        return 26.5 + 0.069 * cells + 0.13 * rows * vp.K + 1.07 * entries < cls + (whole ? 2.7 * entries : 0.0);
    };
    // Joint fill: a vertex without a class digit that can take one of its
    // lookups' vertices in (the structure is described at JointSide).  The
    // digit y with the most configurations.  Classes are kept small -- each
    // end of the three edges has at most one loop dim that the tensor does not
    // map -- so that at most one pair of combined classes belongs to an entry;
    // the dense fill costs two operations per (c, y), this about 100 per
    // configuration and row, so K_i and Ky from 24 up.  uint64 keys: the sums of both
    // vertices' terms must not wrap (fp64 sums past 2^53 round, but never below
    // a key that is exact).
    const bool joint_ok = class_ok && n <= (int)kMaxBacktrackThreads;
    uint32_t joint_key = 3;          // key type of the search (3: not evaluated; 2: none of these fills)
    auto joint_kt = [&] {
        if (joint_key == 3) {
            pase_status kst;
            joint_key = choose_key_type(g, &kst);
            if (kst != PASE_OK) joint_key = 2;
        }
        return joint_key;
    };
    // largest sum of two vertices' terms as keys
    auto joint_top = [&](int i, int j) {
        return ((unsigned __int128)P.qmax[i] + P.qmax[j] + 2) << std::max(P.v[i].bits, P.v[j].bits);
    };
    auto mapped = [&](int e, int u) {   // loop dims of vertex u that edge e's tensor maps
        const auto &d = g->E[e];
        uint32_t m = 0;
        for (uint32_t k = 0; k < d.rank; k++) {
            const int x = (int)d.src == u ? d.src_dim[k] : d.dst_dim[k];
            if (x >= 0) m |= 1u << x;
        }
        return m;
    };
    auto tight = [&](int e) {   // both ends of an edge map all but one of their loop dims
        for (int u : {(int)g->E[e].src, (int)g->E[e].dst})
            if ((uint32_t)__builtin_popcount(mapped(e, u)) + 1 < g->V[u].ndims) return false;
        return true;
    };
    // classes of u's configurations under edge e: the split tuples of the mapped dims
    auto classes_of = [&](int e, int u) {
        const uint32_t m = (uint32_t)__builtin_popcount(mapped(e, u));
        if (!g->factors) {
            uint32_t L = 0, n = 1;
            while ((1u << L) < g->p) L++;
            for (uint32_t k = 1; k <= m; k++) n = n * (L + k) / k;   // C(L + m, m)
            return n;
        }
        // tuples of m factors with product <= q, for every q up to p
        std::vector<uint32_t> cnt(g->p + 1, 1);
        for (uint32_t k = 0; k < m; k++) {
            std::vector<uint32_t> next(g->p + 1, 0);
            for (uint32_t q = 1; q <= g->p; q++)
                for (uint32_t f = 1; f <= q; f++) next[q] += cnt[q / f];
            cnt.swap(next);
        }
        return cnt[g->p];
    };
    // With y's classes fixed, v_i's and v_j's configurations each have one free
    // dim; unless the edge between them ties the two together, all pairs of
    // them that share a class share the combined classes.
    auto one_pair = [&](int eo, int ei, int ey, int vi, int vj) {
        const uint32_t fi = ((1u << g->V[vi].ndims) - 1) & ~mapped(ei, vi);
        const uint32_t fj = ((1u << g->V[vj].ndims) - 1) & ~mapped(ey, vj);
        const auto &d = g->E[eo];
        for (uint32_t k = 0; k < d.rank; k++) {
            const int a = (int)d.src == vi ? d.src_dim[k] : d.dst_dim[k], b = (int)d.src == vi ? d.dst_dim[k] : d.src_dim[k];
            if (a >= 0 && b >= 0 && (fi >> a & 1u) && (fj >> b & 1u)) return false;
        }
        return true;
    };
    // (the plan in `out`, whose allocations the next vertex reuses)
    auto plan_joint = [&](int i, VPlan &out) {
        VPlan &vp = P.v[i];
        if (!joint_ok || vp.K > kJointMaxK || vp.K < 24 || vp.D.size() < 2) return false;
        auto edge_to = [&](const VPlan &v, int w) {   // the one edge of v to w: its id, -1 none, -2 several
            int at = -1;
            for (int e : v.edges)
                if ((int)g->E[e].src == w || (int)g->E[e].dst == w) at = at == -1 ? e : -2;
            return at;
        };
        auto in = [](const TermRef &t, int w) { return std::count(t.dig.begin(), t.dig.end(), w) > 0; };
        int bj = -1, by = -1;
        uint32_t bcls[4] = {0, 0, 0, 0};
        for (const auto &tj : vp.terms) {
            const VPlan &vj = P.v[tj.j];
            if (!vj.classes || vj.joint >= 0 || vj.K > kJointMaxK || tj.dig.empty()) continue;
            const int eo = edge_to(vj, vp.vi);
            bool looked = eo < 0 || !tight(eo);
            for (const auto &t : vj.terms) looked |= in(t, vp.vi);
            if (looked || joint_kt() == 2 || (joint_kt() == 1 && joint_top(i, tj.j) >> 64)) continue;
            for (int y : tj.dig) {
                const int ey = edge_to(vj, y), ei = edge_to(vp, y);
                bool bad = ey < 0 || !tight(ey) || ei == -2 || (ei >= 0 && !tight(ei)) || g->K[y] > kJointMaxK;
                for (const auto &t : vj.terms) bad |= in(t, y);
                uint32_t ni = 0, nti = 0;
                for (const auto &t : vp.terms)
                    if (t.j != tj.j) { bad |= in(t, y); nti++; }
                for (int e : vp.edges) ni += e != ei;
                if (bad || ni > kJointTerms || nti > kJointTerms || vj.edges.size() - 2 > kJointTerms ||
                    vj.terms.size() > kJointTerms || (ei >= 0 && !one_pair(eo, ei, ey, vp.vi, vj.vi)))
                    continue;
                if (by >= 0 && g->K[y] <= g->K[by]) continue;
                const uint32_t cls[4] = {ei >= 0 ? classes_of(ei, vp.vi) : 0, classes_of(ey, vj.vi), classes_of(eo, vj.vi),
                                         classes_of(eo, vp.vi)};
                if (joint_lds(vp.K, vj.K, cls[3], cls[0], cls[1], ei >= 0) > kJointMaxLds ||
                    half_lds(vj.K, cls[2], cls[1]) > kJointMaxLds)
                    continue;
                std::copy(cls, cls + 4, bcls);
                bj = tj.j;
                by = y;
            }
        }
        if (bj < 0 || g->K[by] < 24) return false;
        const VPlan &vj = P.v[bj];
        // v_j's digits first (the upper ones), the others after them in the
        // order of the largest other lookup; y fastest in the table
        std::vector<int> order;
        int big = -1;
        for (size_t t = 0; t < vp.terms.size(); t++)
            if (vp.terms[t].j != bj && (big < 0 || P.v[vp.terms[t].j].N > P.v[vp.terms[big].j].N)) big = (int)t;
        if (big >= 0)
            for (int u : P.v[vp.terms[big].j].layout)
                if (u != vp.vi) order.push_back(u);
        for (int u : vp.D)
            if (std::find(order.begin(), order.end(), u) == order.end()) order.push_back(u);
        const auto has = [](const std::vector<int> &v, int u) { return std::find(v.begin(), v.end(), u) != v.end(); };
        std::vector<int> R;
        uint64_t jupper = 1;
        for (int u : order)
            if (u != by && has(vj.D, u)) { R.push_back(u); jupper *= g->K[u]; }
        for (int u : order)
            if (u != by && !has(vj.D, u)) R.push_back(u);
        out = vp;
        out.jupper = jupper;
        out.R = R;
        out.joint = bj;
        std::copy(bcls, bcls + 4, out.jcls);
        out.z = by;
        out.O.clear();
        out.MO = 1;
        out.MR = vp.N / g->K[by];
        out.TZ = 0;
        out.TM = 1;
        out.nsplit = 1;
        out.cper = vp.K;
        out.parts = 2;
        out.layout = out.R;
        out.layout.push_back(by);
        out.stride.assign(out.layout.size(), 1);
        for (int k = (int)out.layout.size() - 2; k >= 0; k--) out.stride[k] = out.stride[k + 1] * g->K[out.layout[k + 1]];
        out.est_us = 6.0 + (double)out.MR * (1.2e-3 + 1.5e-5 * out.K);
        return true;
    };
    // A column-less vertex without edges (its lookups alone) takes the class
    // kernel's plain minimum while its lookups fit the 32 MB of L2: no prep
    // launch (26 -> 17 us at 3.3e6 cells).  Past that the row kernel's stream
    // is the faster one (80 + 5 against 93 us at 1.8e7 cells, 145 + 5 against
    // 175 at 3.0e7).
    auto stream_small = [&](const VPlan &vp) {
        uint64_t looked = 0;
        for (const auto &t : vp.terms) looked += P.v[t.j].N * 8;
        return vp.edges.empty() && looked <= (32ull << 20);
    };
    VPlan jointp;
    auto plan_one = [&](int i, uint32_t ftz, uint32_t ftm, bool no_split) {
        VPlan &vp = P.v[i];
        vp.classes = vp.exch = false;
        vp.joint = -1;
        const uint32_t tile_cols = ftz ? ftz : g->tile_cols, tile_rows = ftm ? ftm : g->tile_rows;
        // small vertices: the direct fill (one launch, no prep blocks), whose
        // time is a launch plus the gather of every term of every cell
        if (!ftz && g->direct_cells && kernel_mode == 0 && vp.N * vp.K <= g->direct_cells && (g->schedule == kSchedSeq || level_small[vp.level])) {
            vp.kernel = kDirect;
            if (plan_class(i, true)) return;
            vp.est_us = 4.0 + (double)vp.N * vp.K * (1.0 + vp.edges.size() + vp.terms.size()) / 4e5;
            vp.layout = gather_layout(vp);
            vp.nsplit = 1;
            vp.cper = vp.K;
            vp.stride.assign(vp.layout.size(), 1);
            for (int k = (int)vp.layout.size() - 2; k >= 0; k--)
                vp.stride[k] = vp.stride[k + 1] * g->K[vp.layout[k + 1]];
            return;
        }
        // (a small vertex of a level that is not all small: the class kernel
        // still needs no prep launch)
        const bool small = g->direct_cells && vp.N * vp.K <= g->direct_cells;
        const bool cls = !ftz && kernel_mode == 0 && plan_class(i, small);
        if (cls) {
            vp.kernel = small ? kDirect : kRows;
            if (small || !dense_faster(i)) return;
        }
        // the joint fill, unless the dense one below is estimated faster: its
        // rows cost 1.3 ns each at K = 35 (86 us against 27 + 6 us of prep on the
        // three-layer LSTM at p = 16), 8 ns at K = 462 (69 us against 143 + 26 us);
        // a dense fill takes at least 8 us, and its prep as much
        const bool joint = !cls && !ftz && kernel_mode == 0 && plan_joint(i, jointp);
        RowsChoice best;
        // candidates: every digit of D(i) as the column digit z, and -- only
        // when none of those fits -- no column at all (z = -1: every digit is
        // a row digit, each lane streams its own entry's terms over c; for a
        // lookup that covers all of D(i) this reads T_j once, coalesced)
        std::vector<int> zs;
        if (kernel_mode == 0 && vp.D.size() >= 2) zs = vp.D;
        if (kernel_mode == 0 && !vp.D.empty() && !ftz) zs.push_back(-1);
        for (int z : zs) {
            if (z < 0 && best.ok) break;
            {
                RowsChoice rc;
                rc.z = z;
                std::vector<int> O;
                for (const auto &t : vp.terms)
                    if (z >= 0 && t.dig.size() >= 2 && std::count(t.dig.begin(), t.dig.end(), z))
                        for (int u : t.dig)
                            if (u != z) O.push_back(u);
                std::sort(O.begin(), O.end());
                O.erase(std::unique(O.begin(), O.end()), O.end());
                for (int u : vp.D)
                    if (u != z && !std::binary_search(O.begin(), O.end(), u)) rc.R.push_back(u);
                rc.O = O;
                for (int u : rc.O) rc.MO *= g->K[u];
                for (int u : rc.R) rc.MR *= g->K[u];
                if (rc.MR < (z < 0 ? 256u : 16u)) continue;
                uint32_t na = 0;
                for (int u : rc.R) {
                    bool used = false;
                    for (int e : vp.edges) {
                        int other = (int)g->E[e].src == vp.vi ? (int)g->E[e].dst : (int)g->E[e].src;
                        used |= other == u;
                    }
                    for (const auto &t : vp.terms) used |= t.dig.size() == 1 && t.dig[0] == u;
                    na += used;
                }
                bool small = true;   // row terms are read with 32-bit buffer offsets
                double stream_bytes = 0;
                for (const auto &t : vp.terms) {
                    if (t.dig.size() < 2) continue;
                    bool touches = false;
                    for (int u : t.dig) touches |= std::binary_search(rc.R.begin(), rc.R.end(), u);
                    na += touches;
                    if (touches && P.v[t.j].N * 8 >= (1ull << 31)) small = false;
                    if (touches) stream_bytes += 8.0 * (double)std::min<uint64_t>(P.v[t.j].N, vp.N * vp.K);
                }
                if (na > (uint32_t)kMaxATerms || !small) continue;
                rc.na = na;
                const uint32_t Kz = z >= 0 ? g->K[z] : 1;
                const TileChoice tc = tile_choice(rc.MO, rc.MR, z, Kz, vp.K, na, tile_cols, tile_rows, g->tile_parts,
                                                  no_split ? 1u : g->c_splits, stream_bytes);
                rc.ok = tc.ok;
                rc.cost = tc.t.us;
                rc.TZ = tc.TZ;
                rc.TM = tc.TM;
                rc.parts = tc.t.parts;
                rc.nsplit = tc.t.nsplit;
                if (rc.ok && (!best.ok || rc.cost < best.cost)) best = rc;
            }
        }
        if (cls && !(best.ok && best.z >= 0)) return;   // (no column: nothing dense to compare with)
        vp.classes = false;
        if (joint && (!best.ok || jointp.est_us <= std::max(best.cost, 8.0) + 8.0)) {
            std::swap(vp, jointp);
            vp.kernel = kRows;
        } else if (best.ok && best.z < 0 && !ftz && kernel_mode == 0 && stream_small(vp) && plan_class(i, true)) {
            vp.kernel = kRows;
        } else if (best.ok) {
            vp.kernel = kRows;
            vp.z = best.z;
            vp.O = best.O;
            vp.R = best.R;
            vp.MO = best.MO;
            vp.MR = best.MR;
            vp.TZ = best.TZ;
            vp.TM = best.TM;
            vp.na = best.na;
            vp.nchunks = ((vp.z >= 0 ? g->K[vp.z] : 1) + vp.TZ - 1) / vp.TZ;
            vp.ldz = vp.nchunks * vp.TZ;
            vp.layout.clear();
            if (vp.z >= 0) vp.layout.push_back(vp.z);
            vp.layout.insert(vp.layout.end(), vp.O.begin(), vp.O.end());
            vp.layout.insert(vp.layout.end(), vp.R.begin(), vp.R.end());
            vp.parts = best.parts;
            vp.est_us = best.cost;
            const uint64_t ns = best.nsplit;
            vp.cper = (uint32_t)((vp.K + ns - 1) / ns);
            vp.nsplit = (vp.K + vp.cper - 1) / vp.cper;
        } else {
            vp.kernel = kGeneric;
            // gather-bound: ~1e11 cell updates/s, plus a launch's worth of latency
            vp.est_us = 5.0 + (double)vp.N * vp.K / 1e5;
            vp.layout = gather_layout(vp);
            vp.nsplit = 1;
            vp.cper = vp.K;
        }
        vp.stride.assign(vp.layout.size(), 1);
        for (int k = (int)vp.layout.size() - 2; k >= 0; k--)
            vp.stride[k] = vp.stride[k + 1] * g->K[vp.layout[k + 1]];
    };
    // Exchange fill (the structure is described at ExchLookup): i reads one
    // table over all of D(i) = {y, z}, whose vertex j has no edges and only
    // one-digit lookups.  Both of i's edges tight, so that classes are small.
    // Costs ten operations per (c_j, y, z) and two launches, against two per
    // (c_j, c_i, y, z) and three: 660 -> 35 us at K = 84, 462, 462, 462 and
    // 5158 + 1156 -> 115 us at 203, 731, 731, 731; from 24 configurations
    // up, like the joint fill.  With kept tables j's is filled by itself as well.
    auto plan_exchange = [&](int i) {
        VPlan &vp = P.v[i];
        if (!g->fuse_min || !joint_ok || vp.classes || vp.joint >= 0 || vp.kernel == kDirect) return;
        if (vp.terms.size() != 1 || vp.D.size() != 2 || vp.terms[0].dig.size() != 2 || vp.edges.size() != 2 ||
            vp.K < 24 || vp.K > kExchMaxK)
            return;
        const int j = vp.terms[0].j;
        VPlan &vj = P.v[j];
        if (vj.classes || vj.joint >= 0 || vj.kernel == kDirect || !vj.edges.empty() || vj.D.size() != 3 ||
            vj.consumer != i || vj.terms.size() != 3 || vj.K > kClassMaxK)
            return;
        std::vector<int> seen;
        for (const auto &t : vj.terms) {
            if (t.dig.size() != 1 || std::count(seen.begin(), seen.end(), t.dig[0])) return;
            seen.push_back(t.dig[0]);
        }
        for (int u : vp.layout) {
            int k = 0;
            for (int e : vp.edges)
                if ((int)g->E[e].src == u || (int)g->E[e].dst == u) k += tight(e) ? 1 : 2;
            if (k != 1 || g->K[u] > kClassMaxK) return;
        }
        // uint64 keys: sums of a few cases' keys and of the mark of an empty
        // class (2^62) must not wrap
        if (joint_kt() == 2 || (joint_kt() == 1 && joint_top(i, j) >> 60)) return;
        vp.joint = j;
        vp.exch = true;
        // (layout and strides stay those of the dense plan)
        vp.kernel = kRows;
        vp.z = -1;
        vp.O.clear();
        vp.R = vp.layout;
        vp.MO = 1;
        vp.MR = vp.N;
        vp.TZ = 0;
        vp.TM = kExchCols;
        vp.na = 0;
        vp.nsplit = 1;
        vp.cper = vp.K;
        vp.parts = 2;
        // 24 us at 1.8e7 (c, y, z), 102 at 1.1e8
        vp.est_us = 8.0 + 0.9e-6 * (double)vj.K * (double)vp.N;
    };
    for (int i = 0; i < n; i++) {
        plan_one(i, 0, 0, false);
        plan_exchange(i);
    }
    for (int i = 0; i < n; i++) {
        VPlan &vp = P.v[i];
        if (vp.joint < 0) continue;
        vp.jearly = g->schedule != kSchedSeq && g->hoist_elems != 0;
        VPlan &vj = P.v[vp.joint];
        vj.absorbed = i;
        if (g->keep_tables) continue;
        // no fill of its own: what runs in its slot is the half fill (9 us for 84
        // c's of 462 configurations each, 13 for 203 of 731; 9 us for 343 upper
        // indices of 462, 23 for 819 of 731)
        if (vp.exch) {
            vj.kernel = kRows;
            vj.z = vp.vi;
            vj.O.clear();
            vj.MO = 1;
            vj.MR = vp.N;
            vj.TZ = vj.na = vj.parts = 0;
            vj.TM = vj.nsplit = 1;
            vj.cper = vj.K;
            vj.est_us = 8.0 + 4.5e-6 * (double)exch_half_elems(vp.K, vj.K, g->K[vp.layout[0]], g->K[vp.layout[1]]);
        } else {
            vj.est_us = 7.0 + 2e-5 * (double)vp.jupper * vj.K;
        }
    }
    // One launch per level and kernel variant: a small column-form row vertex
    // of a level is re-planned with the tile shape of the level's largest one
    // when its fill then stays under half of that vertex's, so that the two
    // share a launch (the small one's workgroups come first and finish inside
    // the large one's) instead of adding a latency-bound launch of its own.
    // When the largest one is not split over c, the small one is not either:
    // its latency is hidden in the shared launch anyway, and a split would
    // only add the level's reduction launch.
    // Level schedule only: the bulk lane splits a level over two streams.
    if ((g->schedule == kSchedLevel || g->schedule == kSchedSplit) && !g->tile_cols && !g->tile_rows &&
        kernel_mode == 0) {
        std::vector<int> dom((size_t)maxlev + 1, -1);
        for (int i = 0; i < n; i++) {
            const VPlan &vp = P.v[i];
            if (vp.kernel != kRows || vp.z < 0) continue;
            if (vp.absorbed >= 0 && !g->keep_tables) continue;   // not launched
            int &d = dom[vp.level];
            if (d < 0 || vp.est_us > P.v[d].est_us) d = i;
        }
        for (int i = 0; i < n; i++) {
            const int d = dom[P.v[i].level];
            if (d < 0 || d == i || P.v[i].kernel != kRows || P.v[i].z < 0 || P.v[i].joint >= 0) continue;
            if (P.v[i].absorbed >= 0 && !P.v[i].classes && !g->keep_tables) continue;
            // (split chains: only the batched levels share launches level-wide)
            if (g->schedule == kSchedSplit && P.v[i].level >= kSplitBatchedLevels) continue;
            const VPlan &dv = P.v[d];
            if (P.v[i].classes || dv.classes || dv.joint >= 0) {
                // class fills of a batched level share one launch, and with it
                // the largest one's rows per workgroup and use of LDS
                VPlan &ci = P.v[i];
                if (ci.classes && dv.classes && ci.z >= 0 &&
                    class_lds(ci.K, g->K[ci.z], (uint32_t)ci.edges.size() - 1, (uint32_t)ci.terms.size(), dv.lr, true,
                              dv.keep, 512) <= kClassMaxLds) {
                    ci.lr = dv.lr;
                    ci.keep = dv.keep;
                    ci.TM = dv.TM;
                }
                continue;
            }
            const bool unsplit = dv.nsplit == 1 && !g->c_splits;
            if (P.v[i].TZ == dv.TZ && P.v[i].TM == dv.TM && (!unsplit || P.v[i].nsplit == 1)) continue;
            const VPlan saved = P.v[i];
            plan_one(i, dv.TZ, dv.TM, unsplit);
            const VPlan &nv = P.v[i];
            const bool ok = nv.kernel == kRows && nv.z >= 0 && nv.TZ == dv.TZ && nv.TM == dv.TM &&
                            nv.na <= dv.na && nv.est_us <= 0.5 * dv.est_us;
            if (!ok) P.v[i] = saved;
        }
    }
    for (const auto &vp : P.v) {
        if (vp.kernel != kRows || vp.classes || vp.joint >= 0 || (vp.absorbed >= 0 && !g->keep_tables)) continue;
        P.rows_vertices++;
        P.rows_cells += vp.N * vp.K;
        if (vp.z < 0) P.stream_cells += vp.N * vp.K;
    }
    for (auto &vp : P.v) vp.lane = 0;
    if (g->schedule == kSchedBulk) assign_bulk_lanes(P, (double)g->bulk_us);
    if (g->schedule == kSchedSplit) assign_split_lanes(P, (double)g->bulk_us);
    if (g->fuse_min && kernel_mode == 0) fuse_minima(g, P);
    // class tables, one per distinct edge shape (the end u, the other end)
    P.overridden = g->overridden;
    std::vector<int> shape_of(256, -1), shape_next;   // class tables by hash of their map
    auto class_table = [&](int u, int w) {   // of the one edge joining vertices u and w, by u's classes
        for (int e : P.v[std::min(P.pos[u], P.pos[w])].edges) {
            const auto &d = g->E[e];
            const bool is_src = (int)d.src == u;
            if ((is_src ? (int)d.dst : (int)d.src) != w || (!is_src && (int)d.dst != u)) continue;
            DevClassTab t;
            std::memset(&t, 0, sizeof t);
            t.K = g->K[u];
            t.Kz = g->K[w];
            t.ndu = g->V[u].ndims;
            t.ndz = g->V[w].ndims;
            t.rank = d.rank;
            t.factors = g->factors ? 1 : 0;
            uint64_t hash = (t.ndu * 64 + t.ndz) * 64 + t.rank;
            for (uint32_t k = 0; k < kMaxDims; k++) {
                t.udim[k] = (int8_t)(k < d.rank ? (is_src ? d.src_dim[k] : d.dst_dim[k]) : -1);
                t.zdim[k] = (int8_t)(k < d.rank ? (is_src ? d.dst_dim[k] : d.src_dim[k]) : -1);
                hash = hash * 0x9E3779B97F4A7C15ull + (uint64_t)((t.udim[k] + 1) * 16 + t.zdim[k] + 1);
            }
            int &first = shape_of[hash >> 56];
            for (int k = first; k >= 0; k = shape_next[k]) {
                const DevClassTab &o = P.ctabs[k];
                if (o.ndu == t.ndu && o.ndz == t.ndz && o.rank == t.rank &&
                    !std::memcmp(o.udim, t.udim, sizeof t.udim) && !std::memcmp(o.zdim, t.zdim, sizeof t.zdim))
                    return k;
            }
            t.blk0 = P.ctab_blocks;
            P.ctab_blocks += (t.K + t.Kz + 256 / kClassTabLanes - 1) / (256 / kClassTabLanes);
            P.ctabs.push_back(t);
            shape_next.push_back(first);
            return first = (int)P.ctabs.size() - 1;
        }
        return -1;
    };
    for (auto &vp : P.v) {
        if (vp.classes) {
            P.class_fills++;
            if (vp.z >= 0) vp.ctab = class_table(vp.vi, vp.z);
        }
        if (vp.joint >= 0) {
            const int vj = P.v[vp.joint].vi;
            P.joint_fills++;
            if (vp.exch) {
                vp.jtab[0] = class_table(vp.vi, vp.layout[0]);
                vp.jtab[1] = class_table(vp.vi, vp.layout[1]);
                continue;
            }
            vp.jtab[0] = class_table(vp.vi, vp.z);
            vp.jtab[1] = class_table(vj, vp.z);
            vp.jtab[2] = class_table(vj, vp.vi);
            vp.jtab[3] = class_table(vp.vi, vj);
            for (size_t k = 0; k < P.jtabs.size() && vp.jshape < 0; k++)
                if (std::equal(vp.jtab, vp.jtab + 4, P.jtabs[k].tab)) vp.jshape = (int)k;
            if (vp.jshape < 0) {
                DevJointTab t;
                std::memset(&t, 0, sizeof t);
                std::copy(vp.jtab, vp.jtab + 4, t.tab);
                vp.jshape = (int)P.jtabs.size();
                P.jtabs.push_back(t);
            }
        }
    }
    g->stats.plan_ms = ms_since(t1);
    return PASE_OK;
}

// Device memory layout: constant region (configurations, vertex/edge
// descriptors, layer costs, caller-given edge matrices, prep contributions,
// back-substitution descriptors), outputs, the table arenas and scratch.
// Cost tables T_i live from their fill to their single reader (or to the end
// when tables are kept or i is last) and share memory by interval packing;
// argmin tables A_i all live until back-substitution.
enum LayoutMode { kLayoutResident = 0, kLayoutSeq = 1, kLayoutLevel = 2 };
static pase_status layout_memory_mode(pase_graph_t g, LayoutMode mode);

// The bulk lane schedule runs vertices of two streams concurrently and needs
// every table and scratch buffer resident at once; when that exceeds the
// budget, or for the level schedule, tables share memory by lifetimes over
// levels; when even that does not fit, one vertex at a time.
static pase_status layout_memory(pase_graph_t g) {
    const auto t0 = std::chrono::steady_clock::now();
    pase_status st = PASE_ERR_TOO_LARGE;
    if (g->schedule == kSchedBulk || g->schedule == kSchedSplit) st = layout_memory_mode(g, kLayoutResident);
    if (st != PASE_OK && g->schedule != kSchedSeq) st = layout_memory_mode(g, kLayoutLevel);
    if (st != PASE_OK) st = layout_memory_mode(g, kLayoutSeq);
    g->stats.plan_ms += ms_since(t0);
    g->stats.host_plan_ms = g->stats.seq_ms + g->stats.plan_ms;
    return st;
}

static pase_status layout_memory_mode(pase_graph_t g, LayoutMode mode) {
    Plan &P = g->plan;
    // resident: vertices may run in any order the dependencies allow, so
    // every vertex has scratch of its own and no table memory is reused
    const bool resident = mode == kLayoutResident, by_level = mode != kLayoutSeq;
    const uint64_t kb = key_bytes(g);   // bytes per table value and block key
    P.by_level = by_level;
    P.resident = resident;
    P.nslots = 0;
    for (auto &vp : P.v) {
        vp.slot = by_level ? vp.level : (int)(&vp - &P.v[0]);
        P.nslots = std::max(P.nslots, vp.slot + 1);
        vp.prep_after = -2;
    }
    P.hoisted = 0;
    if (mode == kLayoutLevel) hoist_preps(g, P, false);
    if (resident && (g->schedule == kSchedBulk || g->schedule == kSchedSplit)) hoist_preps(g, P, true);
    const int n = (int)P.v.size();
    const uint64_t A = 256;
    uint64_t off = 0;
    P.off_ex = off;
    for (const auto &rows : g->ex_rows) off += rows.size();   // one row set per dimension count
    off = align_up(off, A);
    P.off_vert = off;
    off = align_up(off + g->V.size() * sizeof(DevVertex), A);
    P.off_edge = off;
    off = align_up(off + std::max<size_t>(1, g->E.size()) * sizeof(DevEdge), A);
    P.off_L = off;
    uint64_t sumK = 0;
    for (uint32_t k : g->K) sumK += k;
    off = align_up(off + sumK * 8, A);
    P.off_lsum = off;
    off = align_up(off + sumK, A);
    P.sig_count = 0;
    for (const auto &d : g->E) P.sig_count += (uint64_t)g->K[d.src] + g->K[d.dst];
    P.off_sig = off;
    off = align_up(off + P.sig_count * 8, A);
    P.off_ovedge = off;
    if (g->overridden) off = align_up(off + g->ov_edge.size() * 8, A);
    // contributions: count per vertex (layer + edges + lookups is an upper bound)
    uint64_t ncontrib = 0;
    for (const auto &vp : P.v) ncontrib += 1 + vp.edges.size() + vp.terms.size();
    P.contrib_count = ncontrib;
    P.off_contrib = off;
    off = align_up(off + ncontrib * sizeof(Contrib), A);
    P.off_bt = off;
    off = align_up(off + n * sizeof(BacktrackDesc), A);
    // launch descriptors: only those that some launch reads (all kinds for all
    // vertices were 4 KB a vertex, half of the upload)
    std::fill(std::begin(P.ndesc), std::end(P.ndesc), 0u);
    for (auto &vp : P.v) {
        const bool lazy = vp.absorbed >= 0 && !g->keep_tables;   // (evaluated with the terms of a class fill)
        const bool dense = !vp.classes && vp.joint < 0 && vp.kernel != kDirect && !lazy;
        const bool has[kDescKinds] = {dense, dense && vp.kernel == kRows, dense && vp.kernel == kGeneric,
                                      dense && vp.kernel == kRows && (vp.nsplit > 1 || vp.fused_from >= 0),
                                      vp.kernel == kDirect && !vp.classes, vp.classes || lazy,
                                      vp.joint >= 0 && !vp.exch, vp.exch};
        for (int k = 0; k < kDescKinds; k++) {
            vp.desc[k] = has[k] ? P.ndesc[k] : ~0u;
            P.ndesc[k] += has[k];
        }
    }
    for (int k = 0; k < kDescKinds; k++) {
        P.off_desc[k] = off;
        off = align_up(off + P.ndesc[k] * kDescBytes[k], A);
    }
    P.off_batch = off;
    off = align_up(off + 3 * (uint64_t)n * sizeof(BatchEntry), A);
    P.off_ctdesc = off;
    off = align_up(off + P.ctabs.size() * sizeof(DevClassTab), A);
    P.off_jtdesc = off;
    off = align_up(off + P.jtabs.size() * sizeof(DevJointTab), A);
    // one zero key: the row term that pads a row-kernel vertex up to the
    // row-term count of the launch it shares (uploaded zeroed with the rest)
    P.off_zero = off;
    off = align_up(off + 8, A);
    P.off_cfg = off;
    off = align_up(off + g->V.size() * 4, A);
    P.off_out = off;
    off = align_up(off + sizeof(SearchOut), A);
    // volume transfer model: the edge matrices are computed on the device, so
    // they sit past the uploaded constant region
    P.off_vmat = off;
    if (g->volume && !g->overridden) off = align_up(off + g->mat_total * 8, A);

    // class fills: key-space costs and class tables, written on the device
    P.off_Lk = P.off_fk = P.off_ctab = off;
    if (P.class_fills + P.joint_fills) {
        P.off_fk = off = align_up(off + sumK * 8, A);
        P.off_ctab = off = align_up(off + P.sig_count * 8, A);
        for (auto &t : P.ctabs) {
            t.inv_off = off;
            off = align_up(off + t.K * 2, 16);
            t.perm_off = off;
            off = align_up(off + t.K * 2, 16);
            t.first_off = off;
            off = align_up(off + t.K * 2, 16);
            t.zs_off = off;
            off = align_up(off + t.Kz * sizeof(ClassEntry), 16);
            t.zr_off = off;
            off = align_up(off + t.Kz * 4, 16);
        }
        for (auto &t : P.jtabs) {
            t.off_i = off;
            off += P.ctabs[t.tab[3]].K * sizeof(JointIdI);
            t.off_j = off;
            off += P.ctabs[t.tab[2]].K * sizeof(JointIdI);
            t.off_y = off;
            off += P.ctabs[t.tab[1]].Kz * sizeof(JointY);
            for (int k = 0; k < 3; k++) {   // v_i's to v_j, v_i's to y, v_j's to y
                const int tab = t.tab[k == 0 ? 3 : k - 1];
                t.off_start[k] = off;
                off += tab < 0 ? 0 : (P.ctabs[tab].K + 1) * 2;
            }
            t.off_jown = off;
            off = align_up(off + P.ctabs[t.tab[2]].K * 2, 16);
        }
        off = align_up(off, A);
    }

    auto formed = [&](const VPlan &vp) { return vp.absorbed < 0 || g->keep_tables; };
    // T arena: interval packing over launch slots -- a table is written in the
    // slot of its vertex and last read in the slot of its reader
    struct Iv { int i, s, e; uint64_t size; };
    std::vector<Iv> iv;
    for (int i = 0; i < n; i++) {
        // (the reader of a table may be part of a joint fill in a later slot; its own table is not formed)
        const int reader = i == n - 1 ? i : P.v[i].consumer, by = P.v[reader].absorbed;
        int end = (resident || g->keep_tables || i == n - 1) ? P.nslots
                  : std::max(P.v[reader].slot, by >= 0 ? P.v[by].slot : 0);
        // an absorbed vertex's argmin is evaluated after the fills: the tables it looks up stay
        if (by >= 0) end = P.nslots;
        iv.push_back({i, P.v[i].slot, end, formed(P.v[i]) ? align_up(P.v[i].N * kb, A) : A});
    }
    std::vector<int> order(n);
    std::iota(order.begin(), order.end(), 0);
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return iv[a].size > iv[b].size; });
    // placed tables in ascending offset order: the first gap that fits among
    // those whose lifetimes overlap is found in one pass.  (All of them overlap
    // when every table stays: one after the other.)
    std::vector<int> placed;
    placed.reserve(n);
    uint64_t tbytes = 0;
    for (int k : order) {
        if (resident || g->keep_tables) {
            P.v[iv[k].i].T_off = tbytes;
            tbytes += iv[k].size;
            continue;
        }
        uint64_t cand = 0;
        for (int q : placed) {
            if (!(iv[q].s <= iv[k].e && iv[k].s <= iv[q].e)) continue;
            const uint64_t b0 = P.v[iv[q].i].T_off;
            if (cand + iv[k].size <= b0) break;
            cand = std::max(cand, b0 + iv[q].size);
        }
        P.v[iv[k].i].T_off = cand;
        tbytes = std::max(tbytes, cand + iv[k].size);
        auto at = std::upper_bound(placed.begin(), placed.end(), cand,
                                   [&](uint64_t x, int q) { return x < P.v[iv[q].i].T_off; });
        placed.insert(at, k);
    }
    P.T_bytes = tbytes;
    P.off_T = off;
    off = align_up(off + tbytes, A);
    uint64_t abytes = 0;
    for (auto &vp : P.v) { vp.A_off = abytes; abytes += formed(vp) ? align_up(vp.N * 2, A) : A; }
    P.A_bytes = abytes;
    P.off_A = off;
    off = align_up(off + abytes, A);
    // block and split scratch: vertices of one slot get disjoint pieces; slots reuse it
    std::vector<uint64_t> bsum(P.nslots, 0), psum(P.nslots, 0);
    uint64_t bmax = 0, pmax = 0;
    std::vector<VPlan *> hoisted;
    for (auto &vp : P.v) {
        uint64_t e = 0, pb = 0;
        if (vp.joint >= 0) {
            // the half table
            if (vp.exch)
                e = align_up(exch_half_elems(vp.K, P.v[vp.joint].K, align_up(g->K[vp.layout[0]], kExchCols), g->K[vp.layout[1]]), 32);
            else e = align_up(joint_half_elems(vp.K, P.v[vp.joint].K, g->K[vp.z]) * vp.jupper, 32);
        } else if (vp.classes || (vp.absorbed >= 0 && !g->keep_tables)) {
            // no blocks
        } else if (vp.kernel == kRows) {
            e += align_up(vp.MO * vp.K * vp.ldz, 32);
            for (int u : vp.R) e += align_up((uint64_t)vp.K * g->K[u], 32);
            if (vp.nsplit > 1) pb = align_up((uint64_t)vp.nsplit * vp.N * kb, A);
        } else if (vp.kernel == kGeneric) {
            e += align_up(vp.K, 32);
            for (int u : vp.D) e += align_up((uint64_t)vp.K * g->K[u], 32);
        }   // the direct fill needs no prep blocks and no split scratch
        vp.block_elems = e;
        // (the resident layout keeps every vertex's scratch: one slot for all;
        // a fused minimum's blocks are built and read in its producer's slot)
        const int sl = resident ? 0 : vp.fused_from >= 0 ? P.v[vp.fused_from].slot : vp.slot;
        vp.partial_off = psum[sl];
        psum[sl] += pb;
        pmax = std::max(pmax, psum[sl]);
        if (vp.prep_after >= -1 || vp.jearly) {   // hoisted: blocks live from an earlier slot on
            hoisted.push_back(&vp);
            continue;
        }
        vp.block_off = bsum[sl];
        bsum[sl] += align_up(e * kb, A);
        bmax = std::max(bmax, bsum[sl]);
    }
    // hoisted blocks: after every slot's scratch, one piece each
    for (VPlan *vp : hoisted) {
        vp->block_off = bmax;
        bmax += align_up(vp->block_elems * kb, A);
    }
    P.block_bytes = bmax;
    P.off_block = off;
    off = align_up(off + P.block_bytes, A);
    P.partial_bytes = pmax;
    P.off_partial = off;
    off = align_up(off + P.partial_bytes, A);
    // keys of the fused minima: written in the producer's slot, read in the
    // reader's, so not shared with any other scratch
    P.fused_bytes = 0;
    for (auto &vp : P.v)
        if (vp.fused_from >= 0) {
            vp.fkeys_off = P.fused_bytes;
            P.fused_bytes += align_up(vp.N * kb, A);
        }
    P.off_fused = off;
    off = align_up(off + P.fused_bytes, A);
    P.total = off;
    if (P.total > g->mem_budget)
        return fail(g, PASE_ERR_TOO_LARGE, "device memory need exceeds the memory budget");
    return PASE_OK;
}

// Plan (or, with replan, re-plan from the vertex order on) the search: the
// key type that the plans and the current costs need (R10), then the memory
// layout.  A change to or from 128-bit keys re-plans every vertex (such plans
// run on the generic kernel).  OVERFLOW when a cost bound of the recurrence
// passes 64 bits.
static pase_status lay_out(pase_graph_t g);

static pase_status plan_search(pase_graph_t g, bool replan) {
    pase_status st;
    if (replan && (st = build_structure(g)) != PASE_OK) return st;
    if (!replan) g->plan.bounds = -1;   // (other costs)
    // (a plan with class fills reads the model's own costs: caller-given ones
    // need the dense fills, and the other way round)
    if (replan || g->plan.overridden != g->overridden) {
        if (!replan) reset_fills(g->plan);
        g->dense_only = false;
        if ((st = plan_fills(g)) != PASE_OK) return st;
    }
    const uint32_t kt = choose_key_type(g, &st);
    if (st != PASE_OK) return fail(g, st, "a cost bound of the recurrence exceeds 64 bits");
    if ((kt == 2) != g->plan_wide) {
        g->plan_wide = kt == 2;
        reset_fills(g->plan);
        if ((st = plan_fills(g)) != PASE_OK) return st;
    }
    g->plan_key_type = kt;
    return lay_out(g);
}

// The plan again with the dense fills alone (dense), or with all of them.
static pase_status refill(pase_graph_t g, bool dense) {
    if (dense) g->structured_total = g->plan.total;
    g->dense_only = dense;
    reset_fills(g->plan);
    const pase_status st = plan_fills(g);
    return st == PASE_OK ? layout_memory(g) : st;
}

// The memory layout; past the memory budget, that of the dense fills: the
// class, joint and exchange fills keep key-space costs and class tables beside
// the layer costs and signatures, and so need up to half as much again on a
// chain of small vertices (12 kB more per vertex of 462 configurations).
static pase_status lay_out(pase_graph_t g) {
    const pase_status st = layout_memory(g);
    if (st != PASE_ERR_TOO_LARGE || !(g->plan.class_fills + g->plan.joint_fills)) return st;
    return refill(g, true);
}

// Fit the plan to `limit` bytes of workspace where the dense fills do and the
// others do not (a lent workspace, the static one); back to all fills when
// there is room again.
static pase_status fit_plan(pase_graph_t g, uint64_t limit) {
    pase_status st = PASE_OK;
    if (g->dense_only && g->structured_total <= std::min(limit, g->mem_budget)) {
        g->searched = false;
        st = refill(g, false);
    } else if (g->plan.total > limit && g->plan.class_fills + g->plan.joint_fills) {
        g->searched = false;
        st = refill(g, true);
        if (st != PASE_OK || g->plan.total > limit) st = refill(g, false);
    }
    if (st != PASE_OK) g->planned = false;
    return st;
}

extern "C" pase_status pase_enumerate_configs(pase_graph_t g, uint32_t p) {
    if (!g) return PASE_ERR_INVALID_ARGUMENT;
    const bool factors = g->config_set == 1;
    if (factors && (p == 0 || p > 255))
        return fail(g, PASE_ERR_INVALID_ARGUMENT, "p must be in 1..255 with every integer split");
    if (!factors && (p == 0 || (p & (p - 1)) || p > (1u << 16)))
        return fail(g, PASE_ERR_INVALID_ARGUMENT, "p must be a power of two <= 65536");
    g->enumerated = g->planned = g->searched = g->overridden = false;
    g->ov_layer.clear(); g->ov_edge.clear();
    g->p = p;
    g->factors = factors;
    g->volume = g->transfer_opt == 1;
    g->mat_off.assign(g->E.size(), 0);
    g->mat_total = 0;
    g->mat_row0.assign(g->E.size(), 0);
    g->mat_rows = 0;
    if (g->volume) {
        // the device's volume arithmetic needs Q = prod_t s_u(t) * s_v(t) < 2^32:
        // with distinct mapped loop dims per side each product is at most p,
        // otherwise it is bounded by p to the number of mapped tensor dims
        for (size_t e = 0; e < g->E.size(); e++) {
            const pase_edge_desc &d = g->E[e];
            uint32_t ms = 0, md = 0, ns = 0, nd = 0;
            bool distinct = true;
            for (uint32_t t = 0; t < d.rank; t++) {
                if (d.src_dim[t] >= 0) {
                    distinct &= !((ms >> d.src_dim[t]) & 1u);
                    ms |= 1u << d.src_dim[t];
                    ns++;
                }
                if (d.dst_dim[t] >= 0) {
                    distinct &= !((md >> d.dst_dim[t]) & 1u);
                    md |= 1u << d.dst_dim[t];
                    nd++;
                }
            }
            unsigned __int128 q = 1;
            for (uint32_t k = 0; k < (distinct ? 2u : ns + nd); k++) q *= p;
            if (q >= ((unsigned __int128)1 << 32))
                return fail(g, PASE_ERR_INVALID_ARGUMENT,
                            "volume model: tensor dims mapped to one loop dim make the device fractions too fine");
        }
    }
    const size_t nv = g->V.size();
    g->K.assign(nv, 0);
    g->ex.assign(nv, nullptr);
    g->weight_n.assign(nv, 0);
    g->halo = g->halo_opt == 1;
    g->halo_n.assign(nv, {});
    g->flops.assign(nv, 0);
    g->keep_n.assign(nv, 0);
    g->maxL.assign(nv, 0);
    // the configurations of a vertex depend only on its dimension count
    std::vector<std::vector<uint8_t>> &by_dims = g->ex_rows;
    by_dims.assign(kMaxDims + 1, {});
    for (size_t v = 0; v < nv; v++) {
        const uint32_t d = g->V[v].ndims;
        std::vector<uint8_t> &rows = by_dims[d];
        if (rows.empty()) {
            // split tuples with product <= p in lexicographic order (dim 0
            // slowest), by the lexicographic successor: step the last dim whose
            // next factor (x2, or +1 with every integer) still fits beside the
            // dims before it, and reset the dims after it to 1
            std::vector<uint32_t> cur(d, 1);
            uint64_t cnt = 0;
            for (;;) {
                if (++cnt > 65535) return fail(g, PASE_ERR_TOO_LARGE, "more than 65535 configurations");
                for (uint32_t x : cur) {
                    uint32_t code = x;
                    if (!factors) for (code = 0; (1u << code) < x; code++) {}
                    rows.push_back((uint8_t)code);
                }
                uint64_t prefix[kMaxDims + 1];
                prefix[0] = 1;
                for (uint32_t k = 0; k < d; k++) prefix[k + 1] = prefix[k] * cur[k];
                int k = (int)d - 1;
                for (; k >= 0; k--) {
                    const uint64_t next = factors ? cur[k] + 1ull : 2ull * cur[k];
                    if (prefix[k] * next <= p) break;
                }
                if (k < 0) break;
                cur[k] = factors ? cur[k] + 1 : 2 * cur[k];
                for (uint32_t j = k + 1; j < d; j++) cur[j] = 1;
            }
        }
        uint64_t K = rows.size() / d;
        if (K > 65535) return fail(g, PASE_ERR_TOO_LARGE, "more than 65535 configurations");
        g->K[v] = (uint32_t)K;
        g->ex[v] = &rows;
        uint64_t fl = g->V[v].flops_per_point, keep = 1;
        for (uint32_t k = 0; k < d; k++) {
            if (!mul_ok(fl, g->V[v].size[k], &fl))
                return fail(g, PASE_ERR_OVERFLOW, "layer FLOPs exceed 64 bits");
            if (!((g->V[v].reduce_mask >> k) & 1u) && !mul_ok(keep, g->V[v].size[k], &keep))
                return fail(g, PASE_ERR_OVERFLOW, "layer size exceeds 64 bits");
        }
        if (fl >> 62 || keep >> 62) return fail(g, PASE_ERR_OVERFLOW, "layer cost exceeds 2^62");
        g->flops[v] = fl;
        g->keep_n[v] = keep;
        // t_l <= flops + r * (p - 1) * keep (+ r * 2 * weight words with the gradient term)
        uint64_t comm, m;
        if (!mul_ok(g->r, (uint64_t)(p - 1), &comm) || !mul_ok(comm, keep, &comm) || !add_ok(fl, comm, &m))
            return fail(g, PASE_ERR_OVERFLOW, "layer cost exceeds 64 bits");
        if (g->grad_opt && g->V[v].weight_mask && g->V[v].weight_per_point) {
            uint64_t w = g->V[v].weight_per_point, gr;
            for (uint32_t k = 0; k < d; k++)
                if (((g->V[v].weight_mask >> k) & 1u) && !mul_ok(w, g->V[v].size[k], &w))
                    return fail(g, PASE_ERR_OVERFLOW, "weight tensor exceeds 64 bits");
            if (w >> 60 || !mul_ok(g->r, 2 * w, &gr) || !add_ok(m, gr, &m))
                return fail(g, PASE_ERR_OVERFLOW, "layer cost exceeds 64 bits");
            g->weight_n[v] = w;
        }
        g->halo_n[v].fill(0);
        if (g->halo) {
            // halo term: per halo dim k, I_k = prod of the other input dims'
            // sizes; t_l grows by at most r * 2 * halo[k] * I_k per dim
            const pase_vertex_desc &vd = g->V[v];
            for (uint32_t k = 0; k < d; k++) {
                if (!vd.halo[k]) continue;
                uint64_t I = 1, hw;
                for (uint32_t j = 0; j < d; j++)
                    if (j != k && ((vd.input_mask >> j) & 1u) && !mul_ok(I, vd.size[j], &I))
                        return fail(g, PASE_ERR_OVERFLOW, "input tensor exceeds 64 bits");
                if (I >> 62 || !mul_ok(2ull * vd.halo[k], I, &hw) || !mul_ok(g->r, hw, &hw) || !add_ok(m, hw, &m))
                    return fail(g, PASE_ERR_OVERFLOW, "layer cost exceeds 64 bits");
                g->halo_n[v][k] = I;
            }
        }
        g->maxL[v] = m;
    }
    g->maxR.assign(g->E.size(), 0);
    for (size_t e = 0; e < g->E.size(); e++) {
        // the volume model moves at most the whole tensor in each direction
        const uint64_t words = g->E[e].elems * (g->volume ? 2 : 1);
        if (g->E[e].elems >> 61 || !mul_ok(g->r, words, &g->maxR[e]))
            return fail(g, PASE_ERR_OVERFLOW, "transfer cost exceeds 64 bits");
        if (g->volume) {
            g->mat_off[e] = g->mat_total;
            g->mat_total += (uint64_t)g->K[g->E[e].src] * g->K[g->E[e].dst];
            g->mat_row0[e] = g->mat_rows;
            g->mat_rows += g->K[g->E[e].src];
        }
    }
    g->enumerated = true;
    g->plan_wide = false;
    const pase_status st = plan_search(g, true);
    if (st != PASE_OK) { g->enumerated = false; return st; }
    g->planned = true;
    return PASE_OK;
}

extern "C" pase_status pase_num_configs(pase_graph_t g, uint32_t v, uint32_t *k) {
    if (!g || !k) return PASE_ERR_INVALID_ARGUMENT;
    if (!g->enumerated) return fail(g, PASE_ERR_BAD_STATE, "configurations not enumerated");
    if (v >= g->V.size()) return fail(g, PASE_ERR_INVALID_ARGUMENT, "vertex id out of range");
    *k = g->K[v];
    return PASE_OK;
}

extern "C" pase_status pase_config_splits(pase_graph_t g, uint32_t v, uint32_t idx, uint32_t *splits) {
    if (!g || !splits) return PASE_ERR_INVALID_ARGUMENT;
    if (!g->enumerated) return fail(g, PASE_ERR_BAD_STATE, "configurations not enumerated");
    if (v >= g->V.size() || idx >= g->K[v]) return fail(g, PASE_ERR_INVALID_ARGUMENT, "bad id");
    const uint32_t d = g->V[v].ndims;
    for (uint32_t k = 0; k < d; k++) {
        const uint32_t x = (*g->ex[v])[(size_t)idx * d + k];
        splits[k] = g->factors ? x : 1u << x;
    }
    return PASE_OK;
}

extern "C" pase_status pase_get_sequence(pase_graph_t g, uint32_t *order) {
    if (!g || !order) return PASE_ERR_INVALID_ARGUMENT;
    if (!g->planned) return fail(g, PASE_ERR_BAD_STATE, "configurations not enumerated");
    for (size_t i = 0; i < g->plan.seq.size(); i++) order[i] = (uint32_t)g->plan.seq[i];
    return PASE_OK;
}

extern "C" pase_status pase_get_dependent_set(pase_graph_t g, uint32_t v, uint32_t *out, uint32_t cap,
                                              uint32_t *n) {
    if (!g || !n || (cap && !out)) return PASE_ERR_INVALID_ARGUMENT;
    if (!g->planned) return fail(g, PASE_ERR_BAD_STATE, "configurations not enumerated");
    if (v >= g->V.size()) return fail(g, PASE_ERR_INVALID_ARGUMENT, "vertex id out of range");
    const auto &D = g->plan.v[g->plan.pos[v]].D;
    if (D.size() > cap) return fail(g, PASE_ERR_TOO_LARGE, "output array too small");
    for (size_t k = 0; k < D.size(); k++) out[k] = (uint32_t)D[k];
    *n = (uint32_t)D.size();
    return PASE_OK;
}

extern "C" pase_status pase_set_option(pase_graph_t g, pase_option opt, uint64_t value) {
    if (!g) return PASE_ERR_INVALID_ARGUMENT;
    switch (opt) {
    case PASE_OPT_KEEP_TABLES: g->keep_tables = value != 0; break;
    case PASE_OPT_MEMORY_BUDGET: g->mem_budget = value; break;
    case PASE_OPT_KERNEL:
        if (value > 1) return fail(g, PASE_ERR_INVALID_ARGUMENT, "kernel mode 0 or 1");
        g->kernel_mode = (int)value;
        break;
    case PASE_OPT_KEY_TYPE:
        if (value > 2) return fail(g, PASE_ERR_INVALID_ARGUMENT, "key type 0, 1 or 2");
        g->key_mode = (int)value;
        break;
    case PASE_OPT_PROFILE:
        if (value > 2) return fail(g, PASE_ERR_INVALID_ARGUMENT, "profile 0, 1 or 2");
        g->profile = (int)value;
        break;
    case PASE_OPT_SCHEDULE:
        if (value != kSchedLevel && value != kSchedSeq && value != kSchedBulk && value != kSchedSplit)
            return fail(g, PASE_ERR_INVALID_ARGUMENT, "schedule 0, 1, 4 or 5");
        g->schedule = (int)value;
        break;
    case PASE_OPT_TILE_COLS:
        if (value != 0 && std::find(std::begin(kTZ), std::end(kTZ), value) == std::end(kTZ))
            return fail(g, PASE_ERR_INVALID_ARGUMENT, "tile columns 0, 8, 12, 14, 16, 24 or 28");
        g->tile_cols = (uint32_t)value;
        break;
    case PASE_OPT_TILE_ROWS:
        if (value > 2) return fail(g, PASE_ERR_INVALID_ARGUMENT, "tile rows 0, 1 or 2");
        g->tile_rows = (uint32_t)value;
        break;
    case PASE_OPT_TILE_PARTS:
        if (value != 0 && value != 1 && value != 2 && value != 4)
            return fail(g, PASE_ERR_INVALID_ARGUMENT, "tile parts 0, 1, 2 or 4");
        g->tile_parts = (uint32_t)value;
        break;
    case PASE_OPT_ORDER:
        if (value > 1) return fail(g, PASE_ERR_INVALID_ARGUMENT, "order 0 or 1");
        g->order_mode = (int)value;
        break;
    case PASE_OPT_DIRECT_CELLS:
        g->direct_cells = value;
        break;
    case PASE_OPT_BULK_US:
        if (value > 1000000000ull) return fail(g, PASE_ERR_INVALID_ARGUMENT, "bulk threshold <= 1e9 us");
        g->bulk_us = (uint32_t)value;
        break;
    case PASE_OPT_HALO:
        if (value > 1) return fail(g, PASE_ERR_INVALID_ARGUMENT, "halo 0 or 1");
        g->halo_opt = (uint32_t)value;
        break;
    case PASE_OPT_GRAD_SYNC:
        if (value > 1) return fail(g, PASE_ERR_INVALID_ARGUMENT, "grad sync 0 or 1");
        g->grad_opt = (uint32_t)value;
        break;
    case PASE_OPT_TRANSFER:
        if (value > 1) return fail(g, PASE_ERR_INVALID_ARGUMENT, "transfer model 0 or 1");
        g->transfer_opt = (uint32_t)value;
        break;
    case PASE_OPT_CONFIG_SET:
        if (value > 1) return fail(g, PASE_ERR_INVALID_ARGUMENT, "config set 0 or 1");
        g->config_set = (uint32_t)value;
        break;
    case PASE_OPT_C_SPLITS:
        if (value > 65535) return fail(g, PASE_ERR_INVALID_ARGUMENT, "c splits 0..65535");
        g->c_splits = (uint32_t)value;
        break;
    case PASE_OPT_FUSED_MIN:
        if (value > 1) return fail(g, PASE_ERR_INVALID_ARGUMENT, "fused minimum 0 or 1");
        g->fuse_min = value != 0;
        break;
    case PASE_OPT_HOIST_ELEMS:
        g->hoist_elems = value;
        break;
    default: return fail(g, PASE_ERR_INVALID_ARGUMENT, "unknown option");
    }
    // options that change the plan need a fresh enumeration
    if ((opt == PASE_OPT_KEEP_TABLES || opt == PASE_OPT_KERNEL || opt == PASE_OPT_MEMORY_BUDGET ||
         opt == PASE_OPT_SCHEDULE || opt == PASE_OPT_TILE_COLS || opt == PASE_OPT_TILE_ROWS ||
         opt == PASE_OPT_TILE_PARTS || opt == PASE_OPT_C_SPLITS || opt == PASE_OPT_ORDER ||
         opt == PASE_OPT_DIRECT_CELLS || opt == PASE_OPT_BULK_US || opt == PASE_OPT_KEY_TYPE ||
         opt == PASE_OPT_FUSED_MIN || opt == PASE_OPT_HOIST_ELEMS) &&
        g->enumerated) {
        g->searched = false;
        const pase_status st = plan_search(g, true);
        g->planned = st == PASE_OK;
        if (st != PASE_OK) return st;
    }
    return PASE_OK;
}

extern "C" pase_status pase_override_costs(pase_graph_t g, const uint64_t *layer, const uint64_t *edge) {
    if (!g || !layer || (!edge && !g->E.empty())) return PASE_ERR_INVALID_ARGUMENT;
    if (!g->planned) return fail(g, PASE_ERR_BAD_STATE, "configurations not enumerated");
    const size_t nv = g->V.size(), ne = g->E.size();
    std::vector<uint64_t> old_layer = g->ov_layer, old_layer_off = g->ov_layer_off, old_edge = g->ov_edge,
                          old_edge_off = g->ov_edge_off;
    const bool was = g->overridden;
    g->ov_layer_off.assign(nv, 0);
    uint64_t tot = 0;
    for (size_t v = 0; v < nv; v++) { g->ov_layer_off[v] = tot; tot += g->K[v]; }
    g->ov_layer.assign(layer, layer + tot);
    g->ov_edge_off.assign(ne, 0);
    tot = 0;
    for (size_t e = 0; e < ne; e++) {
        g->ov_edge_off[e] = tot;
        tot += (uint64_t)g->K[g->E[e].src] * g->K[g->E[e].dst];
    }
    g->ov_edge.assign(edge ? edge : layer, edge ? edge + tot : layer);
    g->overridden = true;
    g->searched = false;
    const pase_status st = plan_search(g, false);
    if (st != PASE_OK) {
        // back to the plan of the costs before this call (which was valid)
        const std::string msg = g->err;
        g->overridden = false;
        g->ov_layer.swap(old_layer);
        g->ov_layer_off.swap(old_layer_off);
        g->ov_edge.swap(old_edge);
        g->ov_edge_off.swap(old_edge_off);
        g->overridden = was;
        g->planned = plan_search(g, false) == PASE_OK;
        g->err = msg;
        return st;
    }
    return PASE_OK;
}

extern "C" pase_status pase_workspace_size(pase_graph_t g, uint64_t *bytes) {
    if (!g || !bytes) return PASE_ERR_INVALID_ARGUMENT;
    if (!g->planned) return fail(g, PASE_ERR_BAD_STATE, "configurations not enumerated");
    *bytes = g->plan.total;
    return PASE_OK;
}

extern "C" pase_status pase_set_workspace(pase_graph_t g, void *device_ptr, uint64_t bytes) {
    if (!g) return PASE_ERR_INVALID_ARGUMENT;
    if (device_ptr && ((uintptr_t)device_ptr % 256))
        return fail(g, PASE_ERR_INVALID_ARGUMENT, "workspace must be 256-byte aligned");
    g->lent_ws = device_ptr;
    g->lent_bytes = device_ptr ? bytes : 0;
    g->searched = false;
    return PASE_OK;
}

extern "C" pase_status pase_find_best_strategy(pase_graph_t g, void *stream, uint64_t *min_cost,
                                               uint32_t *config_idx) {
    if (!g || !min_cost || !config_idx) return PASE_ERR_INVALID_ARGUMENT;
    if (!g->planned) return fail(g, PASE_ERR_BAD_STATE, "configurations not enumerated");
    const pase_status st = fit_plan(g, g->lent_ws ? g->lent_bytes : g->mem_budget);
    if (st != PASE_OK) return st;
    if (g->lent_ws && g->lent_bytes < g->plan.total)
        return fail(g, PASE_ERR_OUT_OF_MEMORY, "lent workspace smaller than pase_workspace_size");
    return device_search(g, stream, min_cost, config_idx);
}

extern "C" pase_status pase_plan_check(pase_graph_t g, uint64_t *image_bytes) {
    if (!g || !image_bytes) return PASE_ERR_INVALID_ARGUMENT;
    if (!g->planned) return fail(g, PASE_ERR_BAD_STATE, "configurations not enumerated");
    return plan_check(g, image_bytes);
}

extern "C" pase_status pase_find_best_strategy_noalloc(pase_graph_t g, void *stream, uint64_t *min_cost,
                                                       uint32_t *config_idx) {
    if (!g || !min_cost || !config_idx) return PASE_ERR_INVALID_ARGUMENT;
    if (!g->planned) return fail(g, PASE_ERR_BAD_STATE, "configurations not enumerated");
    const pase_status st = fit_plan(g, PASE_NOALLOC_WORKSPACE_BYTES);
    if (st != PASE_OK) return st;
    return device_search_noalloc(g, stream, min_cost, config_idx);
}

static pase_status find_entry(pase_graph_t g, uint32_t v, const uint32_t *dep_cfg, int *pos,
                              uint64_t *idx) {
    if (!g->searched) return fail(g, PASE_ERR_BAD_STATE, "no search has run");
    if (v >= g->V.size()) return fail(g, PASE_ERR_INVALID_ARGUMENT, "vertex id out of range");
    const VPlan &vp = g->plan.v[g->plan.pos[v]];
    uint64_t x = 0;
    for (size_t k = 0; k < vp.layout.size(); k++) {
        size_t at = std::lower_bound(vp.D.begin(), vp.D.end(), vp.layout[k]) - vp.D.begin();
        uint32_t c = dep_cfg[at];
        if (c >= g->K[vp.layout[k]]) return fail(g, PASE_ERR_INVALID_ARGUMENT, "config out of range");
        x += c * vp.stride[k];
    }
    *pos = g->plan.pos[v];
    *idx = x;
    return PASE_OK;
}

extern "C" pase_status pase_table_entry(pase_graph_t g, uint32_t v, const uint32_t *dep_cfg,
                                        uint64_t *cost, uint32_t *argmin) {
    if (!g || !cost || !argmin) return PASE_ERR_INVALID_ARGUMENT;
    if (v < g->V.size() && g->planned && !g->plan.v[g->plan.pos[v]].D.empty() && !dep_cfg)
        return PASE_ERR_INVALID_ARGUMENT;
    int pos;
    uint64_t idx;
    pase_status st = find_entry(g, v, dep_cfg, &pos, &idx);
    if (st != PASE_OK) return st;
    if (!g->keep_tables && pos != (int)g->plan.v.size() - 1)
        return fail(g, PASE_ERR_BAD_STATE, "tables are not kept (PASE_OPT_KEEP_TABLES)");
    return device_table_entry(g, pos, idx, cost, argmin);
}

extern "C" pase_status pase_table_fingerprint(pase_graph_t g, uint32_t v, uint64_t *fp_cost,
                                              uint64_t *fp_arg) {
    if (!g || !fp_cost || !fp_arg) return PASE_ERR_INVALID_ARGUMENT;
    if (!g->searched) return fail(g, PASE_ERR_BAD_STATE, "no search has run");
    if (v >= g->V.size()) return fail(g, PASE_ERR_INVALID_ARGUMENT, "vertex id out of range");
    int pos = g->plan.pos[v];
    if (!g->keep_tables && pos != (int)g->plan.v.size() - 1)
        return fail(g, PASE_ERR_BAD_STATE, "tables are not kept (PASE_OPT_KEEP_TABLES)");
    return device_fingerprint(g, pos, fp_cost, fp_arg);
}

extern "C" pase_status pase_layer_costs(pase_graph_t g, uint32_t v, uint64_t *out) {
    if (!g || !out) return PASE_ERR_INVALID_ARGUMENT;
    if (!g->searched) return fail(g, PASE_ERR_BAD_STATE, "no search has run");
    if (v >= g->V.size()) return fail(g, PASE_ERR_INVALID_ARGUMENT, "vertex id out of range");
    return device_layer_costs(g, v, out);
}

extern "C" pase_status pase_edge_costs(pase_graph_t g, uint32_t e, uint64_t *out) {
    if (!g || !out) return PASE_ERR_INVALID_ARGUMENT;
    if (!g->searched) return fail(g, PASE_ERR_BAD_STATE, "no search has run");
    if (e >= g->E.size()) return fail(g, PASE_ERR_INVALID_ARGUMENT, "edge id out of range");
    return device_edge_costs(g, e, out);
}

extern "C" pase_status pase_stats(pase_graph_t g, pase_run_stats *out) {
    if (!g || !out) return PASE_ERR_INVALID_ARGUMENT;
    if (!g->searched) return fail(g, PASE_ERR_BAD_STATE, "no search has run");
    *out = g->stats;
    return PASE_OK;
}

extern "C" pase_status pase_vertex_info_get(pase_graph_t g, uint32_t v, pase_vertex_info *out) {
    if (!g || !out) return PASE_ERR_INVALID_ARGUMENT;
    if (!g->planned) return fail(g, PASE_ERR_BAD_STATE, "configurations not enumerated");
    if (v >= g->V.size()) return fail(g, PASE_ERR_INVALID_ARGUMENT, "vertex id out of range");
    const VPlan &vp = g->plan.v[g->plan.pos[v]];
    pase_vertex_info x;
    std::memset(&x, 0, sizeof x);
    x.position = (uint32_t)g->plan.pos[v];
    x.kernel = (uint32_t)vp.kernel;
    x.num_configs = vp.K;
    x.dep_count = (uint32_t)vp.D.size();
    x.entries = vp.N;
    x.cells = vp.N * vp.K;
    x.column = vp.kernel == kRows ? vp.z : -1;
    x.outer = (uint32_t)vp.MO;
    x.rows = (uint32_t)vp.MR;
    x.tile_cols = vp.TZ;
    x.tile_rows = vp.TM;
    x.parts = vp.kernel == kRows ? vp.parts : 0;
    x.splits = vp.absorbed >= 0 && !g->keep_tables ? 0 : vp.nsplit;
    x.row_terms = vp.na;
    x.lookups = (uint32_t)vp.terms.size();
    x.fill_ms = vp.fill_ms;
    x.level = (uint32_t)vp.level;
    x.lane = (uint32_t)vp.lane;
    if (cost_bounds(g)) {
        x.key_bound = g->plan.qmax[x.position];
        x.table_bound = g->plan.tmax[x.position];
    } else {
        x.key_bound = x.table_bound = ~0ull;
    }
    x.key_type = g->plan_key_type;
    x.fused = vp.fuse_into >= 0 || (vp.absorbed >= 0 && g->plan.v[vp.absorbed].exch) ? 1u
              : vp.fused_from >= 0 || vp.exch ? 2u : 0u;
    x.prep_after = vp.prep_after;
    x.prep_lane = (uint32_t)vp.prep_lane;
    *out = x;
    return PASE_OK;
}
