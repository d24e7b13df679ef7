// Host planning of one search's launches (no HIP calls, so that it runs and
// is checked without a GPU): kernel descriptors of every position resolved
// against the workspace base, the batched launches of each launch slot, and
// the constant-region image the device runtime uploads before the first
// kernel.
#include <algorithm>
#include <cstring>
#include <map>
#include <type_traits>

#include "launch.h"

namespace pase {

static uint32_t grid_for(uint64_t n, uint32_t block = 256, uint32_t cap = 8192) {
    uint64_t b = (n + block - 1) / block;
    return (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>(b, cap));
}

static uint32_t plan_digit(const VPlan &vp, int vertex) {
    for (size_t k = 0; k < vp.layout.size(); k++)
        if (vp.layout[k] == vertex) return (uint32_t)k;
    return ~0u;
}

// Strides with which consumer position i reads table T_j: (stride of v_i, per plan digit).
static void lookup_strides(const Plan &P, int i, int j, uint32_t &sc, uint32_t sd[kMaxDep]) {
    const VPlan &vi = P.v[i], &vj = P.v[j];
    sc = 0;
    for (int k = 0; k < kMaxDep; k++) sd[k] = 0;
    for (size_t k = 0; k < vj.layout.size(); k++) {
        int u = vj.layout[k];
        if (u == vi.vi) sc = (uint32_t)vj.stride[k];
        else sd[plan_digit(vi, u)] = (uint32_t)vj.stride[k];
    }
}

// Largest element index a strided read can reach: (K-1)*sc + sum (radix-1)*stride.
static uint64_t max_index(uint32_t K, uint32_t sc, const uint32_t *sd, const uint32_t *rad, int m) {
    uint64_t x = (uint64_t)(K - 1) * sc;
    for (int k = 0; k < m; k++) x += (uint64_t)(rad[k] - 1) * sd[k];
    return x;
}

template <typename KeyT>
pase_status build_launches(pase_graph_t g, char *ws, std::vector<Launch<KeyT>> &out,
                           std::vector<Contrib> &contrib) {
    const Plan &P = g->plan;
    const int n = (int)P.v.size();
    out.clear();
    out.resize(n);
    contrib.clear();
    const uint64_t *ovedge = (const uint64_t *)(ws + P.off_ovedge);
    // element offsets of every vertex's layer costs and every edge's signatures
    std::vector<uint64_t> koff(g->V.size() + 1, 0), soff(g->E.size() + 1, 0);
    for (size_t v = 0; v < g->V.size(); v++) koff[v + 1] = koff[v] + g->K[v];
    for (size_t e = 0; e < g->E.size(); e++) soff[e + 1] = soff[e] + g->K[g->E[e].src] + g->K[g->E[e].dst];
    for (int i = 0; i < n; i++) {
        const VPlan &vp = P.v[i];
        Launch<KeyT> &L = out[i];
        KeyT *blocks = (KeyT *)(ws + P.off_block + vp.block_off);
        const bool lazy = vp.absorbed >= 0 && !g->keep_tables && !vp.classes;   // of an exchange fill
        const bool dense = !vp.classes && vp.joint < 0 && vp.kernel != kDirect && !lazy;
        if (dense) std::memset(&L.prep, 0, sizeof L.prep);
        L.prep.blocks = blocks;
        L.prep.vi = (uint32_t)vp.vi;
        L.prep.K = vp.K;
        L.prep.bits = vp.bits;
        uint32_t rad[kMaxDep];
        for (size_t k = 0; k < vp.layout.size(); k++) rad[k] = g->K[vp.layout[k]];
        const int m = (int)vp.layout.size();
        bool bounds_ok = true;
        auto other_of = [&](int e) {
            return (int)g->E[e].src == vp.vi ? (int)g->E[e].dst : (int)g->E[e].src;
        };
        auto edge_contrib = [&](int e, uint32_t dig) {
            Contrib c;
            std::memset(&c, 0, sizeof c);
            bool is_src = (int)g->E[e].src == vp.vi;
            if (g->overridden || g->volume) {
                c.kind = kContribTable;
                c.raw_u64 = 1;
                c.ptr = g->overridden ? ovedge + g->ov_edge_off[e] : (const uint64_t *)(ws + P.off_vmat) + g->mat_off[e];
                uint32_t Kd = g->K[g->E[e].dst];
                if (is_src) { c.sc = Kd; c.sd[dig] = 1; }
                else { c.sc = 1; c.sd[dig] = Kd; }
                if (max_index(vp.K, c.sc, c.sd, rad, m) >= (uint64_t)g->K[g->E[e].src] * Kd)
                    bounds_ok = false;
            } else {
                c.kind = kContribEdge;
                c.edge = (uint32_t)e;
                c.dig = dig;
                c.vi_is_src = is_src;
            }
            contrib.push_back(c);
        };
        auto table_contrib = [&](const TermRef &t) {
            Contrib c;
            std::memset(&c, 0, sizeof c);
            c.kind = kContribTable;
            c.ptr = ws + P.off_T + P.v[t.j].T_off;
            lookup_strides(P, i, t.j, c.sc, c.sd);
            // the prep block only feeds digits of the lookup, so every index stays inside T_j
            if (max_index(vp.K, c.sc, c.sd, rad, m) >= P.v[t.j].N) bounds_ok = false;
            contrib.push_back(c);
        };
        auto layer_contrib = [&]() {
            Contrib c;
            std::memset(&c, 0, sizeof c);
            c.kind = kContribLayer;
            contrib.push_back(c);
        };
        uint64_t boff = 0;
        auto add_block = [&](const std::vector<int> &pre, int post, uint32_t ld, uint32_t cb) -> int {
            Block &bk = L.prep.blk[L.prep.nblocks];
            std::memset(&bk, 0, sizeof bk);
            bk.npre = (uint32_t)pre.size();
            uint64_t el = 1;
            for (size_t k = 0; k < pre.size(); k++) {
                bk.pre[k] = plan_digit(vp, pre[k]);
                bk.prerad[k] = g->K[pre[k]];
                el *= g->K[pre[k]];
            }
            bk.post = post >= 0 ? (int32_t)plan_digit(vp, post) : -1;
            bk.postrad = post >= 0 ? g->K[post] : 1;
            bk.ld = ld;
            bk.elems = el * vp.K * ld;
            bk.out_off = boff;
            boff += (bk.elems + 31) / 32 * 32;
            bk.c_begin = cb;
            bk.c_end = (uint32_t)contrib.size();
            bk.rows = (uint32_t)el;
            // a workgroup covers `span` runs of kPrepThreads elements, so that
            // the chain of scalar loads of the block's descriptors and
            // contributions is paid once per span; large blocks keep at
            // least ~4096 workgroups
            const uint64_t runs = ((uint64_t)vp.K * ld + kPrepThreads - 1) / kPrepThreads;
            bk.span = (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>(8, runs * el / 4096));
            bk.chunks = (uint32_t)((runs + bk.span - 1) / bk.span);
            bk.wg_begin = L.prep.nwg;
            L.prep.nwg += bk.rows * bk.chunks;
            L.prep.total += bk.elems;
            return (int)L.prep.nblocks++;
        };
        // the two ends' element offsets of an edge of vertex `me`: its own, the other's
        auto edge_ends = [&](int e, int me, uint64_t &oc, uint64_t &oo) {
            const bool is_src = (int)g->E[e].src == me;
            const uint64_t s0 = soff[e], d0 = s0 + g->K[g->E[e].src];
            oc = is_src ? s0 : d0;
            oo = is_src ? d0 : s0;
        };
        if (vp.exch) {
            const VPlan &vj = P.v[vp.joint];
            ExchArgs &xa = L.xa;
            std::memset(&xa, 0, sizeof xa);
            const int y = vp.layout[0], z = vp.layout[1];
            const KeyT *fk = (const KeyT *)(ws + P.off_fk), *Lk = (const KeyT *)(ws + P.off_Lk);
            xa.Li = Lk + koff[vp.vi];
            xa.Lj = Lk + koff[vj.vi];
            xa.Ki = vp.K;
            xa.Kj = vj.K;
            xa.Ky = g->K[y];
            xa.Kyp = (xa.Ky + kExchCols - 1) / kExchCols * kExchCols;
            xa.Kz = g->K[z];
            xa.bits = vp.bits;
            xa.out_shift = vp.out_shift;
            xa.shift = (int32_t)vp.bits - (int32_t)vj.bits;
            if (vp.layout.size() != 2 || vp.stride[1] != 1 || vp.stride[0] != xa.Kz || xa.Ki > kExchMaxK)
                return fail(g, PASE_ERR_INTERNAL, "exchange fill layout");
            for (int e : vp.edges) {
                uint64_t oc, oo;
                edge_ends(e, vp.vi, oc, oo);
                const bool to_y = other_of(e) == y;
                if (!to_y && other_of(e) != z) return fail(g, PASE_ERR_INTERNAL, "exchange fill edge");
                (to_y ? xa.f1x : xa.f2x) = fk + oc;
                (to_y ? xa.f1y : xa.f2z) = fk + oo;
            }
            if (!xa.f1x || !xa.f2x || vj.terms.size() != 3 || vp.jtab[0] < 0 || vp.jtab[1] < 0) return fail(g, PASE_ERR_INTERNAL, "exchange fill edges");
            for (const auto &t : vj.terms) {
                const int k = t.dig[0] == vp.vi ? 0 : t.dig[0] == y ? 1 : t.dig[0] == z ? 2 : -1;
                uint32_t sdv[kMaxDep], vrad[kMaxDep];
                if (t.dig.size() != 1 || k < 0 || xa.l[k].ptr) return fail(g, PASE_ERR_INTERNAL, "exchange fill lookup");
                lookup_strides(P, vp.joint, t.j, xa.l[k].sc, sdv);
                for (size_t q = 0; q < vj.layout.size(); q++) {
                    vrad[q] = g->K[vj.layout[q]];
                    if (vj.layout[q] == t.dig[0]) xa.l[k].sd = sdv[q];
                }
                if (max_index(vj.K, xa.l[k].sc, sdv, vrad, (int)vj.layout.size()) >= P.v[t.j].N) bounds_ok = false;
                xa.l[k].ptr = ws + P.off_T + P.v[t.j].T_off;
            }
            const DevClassTab &t1 = P.ctabs[vp.jtab[0]], &t2 = P.ctabs[vp.jtab[1]];
            xa.perm1 = (const uint16_t *)(ws + t1.perm_off);
            xa.first1 = (const uint16_t *)(ws + t1.first_off);
            xa.first2 = (const uint16_t *)(ws + t2.first_off);
            xa.zr1 = (const uint32_t *)(ws + t1.zr_off);
            xa.zr2 = (const uint32_t *)(ws + t2.zr_off);
            xa.half = blocks;
            boff = exch_half_elems(xa.Ki, xa.Kj, xa.Kyp, xa.Kz);
            xa.T = ws + P.off_T + vp.T_off;
            xa.A = (uint16_t *)(ws + P.off_A + vp.A_off);
            xa.nblk = xa.Kyp / kExchCols * ((xa.Kz + 63) / 64);
            xa.lds = (uint32_t)exch_lds(xa.Ki);
            L.joint = true;
        } else if (lazy) {
            // not filled: its terms, for one evaluation
            ClassArgs &ca = L.ca;
            std::memset(&ca, 0, sizeof ca);
            ca.Lk = (const KeyT *)(ws + P.off_Lk) + koff[vp.vi];
            ca.K = vp.K;
            ca.Kz = 1;
            ca.bits = vp.bits;
            ca.rows = 1;
            ca.nR = (uint32_t)vp.layout.size();
            for (size_t k = 0; k < vp.layout.size(); k++) ca.rad[k] = g->K[vp.layout[k]];
            if (!vp.edges.empty() || vp.terms.size() > (size_t)kMaxClassTerms)
                return fail(g, PASE_ERR_INTERNAL, "a vertex without a table");
            for (const auto &t : vp.terms) {
                ClassTerm &ct = ca.t[ca.nt++];
                lookup_strides(P, i, t.j, ct.sc, ct.sd);
                if (max_index(vp.K, ct.sc, ct.sd, rad, m) >= P.v[t.j].N) bounds_ok = false;
                ct.ptr = ws + P.off_T + P.v[t.j].T_off;
            }
        } else if (vp.joint >= 0) {
            if constexpr (sizeof(KeyT) != 8) {
                return fail(g, PASE_ERR_INTERNAL, "joint fill with 128-bit keys");
            } else {
                const VPlan &vj = P.v[vp.joint];
                JointArgs &ja = L.ja;
                std::memset(&ja, 0, sizeof ja);
                const uint64_t *sig = (const uint64_t *)(ws + P.off_sig);
                const KeyT *fk = (const KeyT *)(ws + P.off_fk), *Lk = (const KeyT *)(ws + P.off_Lk);
                auto rest_digit = [&](int u) { return (uint32_t)(std::find(vp.R.begin(), vp.R.end(), u) - vp.R.begin()); };
                ja.Ky = g->K[vp.z];
                ja.bits = vp.bits;
                ja.out_shift = vp.out_shift;
                ja.upper = (uint32_t)vp.jupper;
                ja.lower = (uint32_t)(vp.MR / vp.jupper);
                ja.nR = (uint32_t)vp.R.size();
                for (size_t k = 0; k < vp.R.size(); k++) ja.rad[k] = g->K[vp.R[k]];
                for (int sd = 0; sd < 2; sd++) {
                    const VPlan &v = sd ? vj : vp;
                    JointSide &s = ja.s[sd];
                    const int other = sd ? vp.vi : vj.vi;
                    s.K = v.K;
                    s.shift = (int32_t)vp.bits - (int32_t)v.bits;
                    s.Lk = Lk + koff[v.vi];
                    for (int e : v.edges) {
                        const int u = (int)g->E[e].src == v.vi ? (int)g->E[e].dst : (int)g->E[e].src;
                        uint64_t oc, oo;
                        edge_ends(e, v.vi, oc, oo);
                        if (u == other) {   // (one of v_j's edges: v_j comes first)
                            ja.fj_o = fk + oc;
                            ja.fi_o = fk + oo;
                            continue;
                        }
                        if (u == vp.z) {
                            (sd ? ja.fj_y : ja.fi_y) = fk + oc;
                            (sd ? ja.fj_yy : ja.fi_yy) = fk + oo;
                            continue;
                        }
                        if (s.ne >= kJointTerms || rest_digit(u) >= ja.nR) return fail(g, PASE_ERR_INTERNAL, "joint edges");
                        ClassEdge &ce = s.e[s.ne++];
                        ce.sig_c = sig + oc;
                        ce.sig_o = sig + oo;
                        ce.f_c = fk + oc;
                        ce.f_o = fk + oo;
                        ce.dig = rest_digit(u);
                    }
                    for (const auto &t : v.terms) {
                        if (t.j == vp.joint) continue;
                        if (s.nt >= kJointTerms) return fail(g, PASE_ERR_INTERNAL, "joint lookups");
                        ClassTerm &ct = s.t[s.nt++];
                        // strides by v's plan digits, then by v_i's rest digits
                        uint32_t sdv[kMaxDep], vrad[kMaxDep];
                        lookup_strides(P, sd ? vp.joint : i, t.j, ct.sc, sdv);
                        for (size_t k = 0; k < v.layout.size(); k++) vrad[k] = g->K[v.layout[k]];
                        if (max_index(v.K, ct.sc, sdv, vrad, (int)v.layout.size()) >= P.v[t.j].N) bounds_ok = false;
                        ct.ptr = ws + P.off_T + P.v[t.j].T_off;
                        for (size_t k = 0; k < v.layout.size(); k++) {
                            if (!sdv[k]) continue;
                            const uint32_t r = rest_digit(v.layout[k]);
                            if (r >= ja.nR) return fail(g, PASE_ERR_INTERNAL, "joint lookup digit");
                            ct.sd[r] = sdv[k];
                        }
                    }
                }
                const DevJointTab &jt = P.jtabs[vp.jshape];
                ja.ii = (const JointIdI *)(ws + jt.off_i);
                ja.ij = (const JointIdJ *)(ws + jt.off_j);
                ja.y = (const JointY *)(ws + jt.off_y);
                ja.start_o = (const uint16_t *)(ws + jt.off_start[0]);
                ja.start_yi = (const uint16_t *)(ws + jt.off_start[1]);
                ja.start_yj = (const uint16_t *)(ws + jt.off_start[2]);
                ja.jown = (const uint16_t *)(ws + jt.off_jown);
                ja.jplace = (const uint16_t *)(ws + P.ctabs[vp.jtab[1]].inv_off);
                ja.yi = vp.jcls[0];
                ja.yj = vp.jcls[1];
                ja.oj = vp.jcls[2];
                ja.oi = vp.jcls[3];
                ja.has_e = ja.fi_y != nullptr;
                if (!ja.fj_y || !ja.fi_o) return fail(g, PASE_ERR_INTERNAL, "joint edge");
                ja.half = blocks;
                boff = joint_half_elems(vp.K, vj.K, ja.Ky) * ja.upper;
                ja.T = ws + P.off_T + vp.T_off;
                ja.A = (uint16_t *)(ws + P.off_A + vp.A_off);
                const uint32_t most = std::max(std::max(vp.K, vj.K), ja.Ky);
                // (one configuration per thread up to 768; past that 512 threads with two)
                ja.threads = most <= 768 ? (most + 63) / 64 * 64 : 512;
                if (most > kJointMaxK || (uint64_t)ja.threads * 2 < most) return fail(g, PASE_ERR_INTERNAL, "joint size");
                ja.lds = (uint32_t)joint_lds(vp.K, vj.K, ja.oi, ja.yi, ja.yj, ja.has_e);
                ja.hlds = (uint32_t)half_lds(vj.K, ja.oj, ja.yj);
                if (ja.lds > kJointMaxLds || ja.hlds > kJointMaxLds) return fail(g, PASE_ERR_INTERNAL, "joint fill LDS");
                // segments: about 2048 workgroups (each brings its upper index's half table in), or one per row
                ja.seg = (uint32_t)std::max<uint64_t>(1, std::min<uint64_t>(ja.lower, 2048 / ja.upper));
                ja.nblk = (uint32_t)(((uint64_t)ja.upper * ja.seg + 7) / 8 * 8);
                ja.hblk = std::min<uint32_t>(ja.upper, 1024);
                L.joint = true;
            }
        } else if (vp.classes) {
            if constexpr (sizeof(KeyT) != 8) {
                return fail(g, PASE_ERR_INTERNAL, "class fill with 128-bit keys");
            } else {
                ClassArgs &ca = L.ca;
                std::memset(&ca, 0, sizeof ca);
                ca.Lk = (const KeyT *)(ws + P.off_Lk) + koff[vp.vi];
                ca.K = vp.K;
                ca.Kz = vp.z >= 0 ? g->K[vp.z] : 1;
                ca.has_z = vp.z >= 0;
                ca.bits = vp.bits;
                ca.out_shift = vp.out_shift;
                ca.rows = (uint32_t)vp.MR;
                ca.nR = (uint32_t)vp.R.size();
                for (size_t k = 0; k < vp.R.size(); k++) ca.rad[k] = g->K[vp.R[k]];
                ca.lr = vp.lr;
                ca.keep = vp.keep;
                ca.staged = vp.lr >= kClassStagedRows;
                ca.nblk = (uint32_t)((((vp.MR + (1u << vp.lr) - 1) >> vp.lr) + 7) / 8 * 8);
                const uint64_t *sig = (const uint64_t *)(ws + P.off_sig);
                const KeyT *fk = (const KeyT *)(ws + P.off_fk);
                bool zdone = vp.z < 0;
                for (int e : vp.edges) {
                    uint64_t oc, oo;
                    edge_ends(e, vp.vi, oc, oo);
                    if (g->volume) {   // the edge's matrix as a lookup
                        if (ca.nt >= (uint32_t)kMaxClassTerms) return fail(g, PASE_ERR_INTERNAL, "class lookups");
                        ClassTerm &ct = ca.t[ca.nt++];
                        const uint32_t Kd = g->K[g->E[e].dst];
                        const bool is_src = (int)g->E[e].src == vp.vi;
                        const uint32_t dig = (uint32_t)(std::find(vp.R.begin(), vp.R.end(), other_of(e)) - vp.R.begin());
                        if (dig >= ca.nR) return fail(g, PASE_ERR_INTERNAL, "class edge digit");
                        ct.ptr = (const uint64_t *)(ws + P.off_vmat) + g->mat_off[e];
                        ct.raw = 1;
                        ct.sc = is_src ? Kd : 1;
                        ct.sd[dig] = is_src ? 1 : Kd;
                        continue;
                    }
                    if (other_of(e) == vp.z) {
                        if (zdone || vp.ctab < 0) return fail(g, PASE_ERR_INTERNAL, "class edge");
                        zdone = true;
                        ca.fzc = fk + oc;
                        ca.fzo = fk + oo;
                        ca.sig_zc = sig + oc;
                        ca.sig_zo = sig + oo;
                        ca.inv = (const uint16_t *)(ws + P.ctabs[vp.ctab].inv_off);
                        ca.zs = (const ClassEntry *)(ws + P.ctabs[vp.ctab].zs_off);
                        continue;
                    }
                    if (ca.ne >= (uint32_t)kMaxClassEdges) return fail(g, PASE_ERR_INTERNAL, "class edges");
                    ClassEdge &ce = ca.e[ca.ne++];
                    ce.sig_c = sig + oc;
                    ce.sig_o = sig + oo;
                    ce.f_c = fk + oc;
                    ce.f_o = fk + oo;
                    ce.dig = (uint32_t)(std::find(vp.R.begin(), vp.R.end(), other_of(e)) - vp.R.begin());
                    if (ce.dig >= ca.nR) return fail(g, PASE_ERR_INTERNAL, "class edge digit");
                }
                if (!zdone) return fail(g, PASE_ERR_INTERNAL, "class edge");
                for (const auto &t : vp.terms) {
                    if (ca.nt >= (uint32_t)kMaxClassTerms) return fail(g, PASE_ERR_INTERNAL, "class lookups");
                    ClassTerm &ct = ca.t[ca.nt++];
                    uint32_t sd[kMaxDep];
                    lookup_strides(P, i, t.j, ct.sc, sd);
                    if (max_index(vp.K, ct.sc, sd, rad, m) >= P.v[t.j].N) bounds_ok = false;
                    if (vp.z >= 0 && sd[0]) return fail(g, PASE_ERR_INTERNAL, "class digit in a lookup");
                    ct.ptr = ws + P.off_T + P.v[t.j].T_off;
                    for (size_t k = 0; k < vp.R.size(); k++) ct.sd[k] = sd[(vp.z >= 0 ? 1 : 0) + k];
                }
                ca.T = ws + P.off_T + vp.T_off;
                ca.A = (uint16_t *)(ws + P.off_A + vp.A_off);
                // (the launch's workgroups may be larger than planned: at most 512 threads)
                const uint64_t lds = class_lds(ca.K, ca.Kz, ca.ne, ca.nt, ca.lr, ca.has_z, ca.keep, 512);
                if (lds > kClassMaxLds || (ca.has_z && !ca.keep && ca.lr != 6))
                    return fail(g, PASE_ERR_INTERNAL, "class fill LDS");
                ca.lds = (uint32_t)lds;
                L.cls = true;
            }
        } else if (vp.kernel == kDirect) {
            // every term over all plan digits; no blocks
            DirectArgs &da = L.da;
            std::memset(&da, 0, sizeof da);
            da.c_begin = (uint32_t)contrib.size();
            layer_contrib();
            for (int e : vp.edges) edge_contrib(e, plan_digit(vp, other_of(e)));
            for (const auto &t : vp.terms) table_contrib(t);
            da.c_end = (uint32_t)contrib.size();
            da.vi = (uint32_t)vp.vi;
            da.K = vp.K;
            da.bits = vp.bits;
            da.out_shift = vp.out_shift;
            da.m = (uint32_t)vp.layout.size();
            for (size_t k = 0; k < vp.layout.size(); k++) da.rad[k] = g->K[vp.layout[k]];
            // lanes per entry: enough threads to fill the GPU, at most a
            // workgroup (four waves, combined in LDS), at most K
            da.group_log2 = 0;
            while (da.group_log2 < 8 && (vp.N << da.group_log2) < 65536 && (2u << da.group_log2) <= vp.K)
                da.group_log2++;
            da.N = vp.N;
            da.T = ws + P.off_T + vp.T_off;
            da.A = (uint16_t *)(ws + P.off_A + vp.A_off);
            da.nblk = (uint32_t)std::min<uint64_t>(((vp.N << da.group_log2) + 255) / 256, 65535);
            L.direct = true;
        } else if (vp.kernel == kRows) {
            // column block B over (O..., c, z): everything not touching a row digit
            std::vector<int> OZ = vp.O;
            OZ.push_back(vp.z);
            auto in_oz = [&](int u) { return std::find(OZ.begin(), OZ.end(), u) != OZ.end(); };
            uint32_t cb = (uint32_t)contrib.size();
            layer_contrib();
            for (int e : vp.edges)
                if (in_oz(other_of(e))) edge_contrib(e, plan_digit(vp, other_of(e)));
            for (const auto &t : vp.terms) {
                bool all = true;
                for (int u : t.dig) all &= in_oz(u);
                if (all) table_contrib(t);
            }
            add_block(vp.O, vp.z, vp.ldz, cb);
            RowsArgs &ra = L.ra;
            std::memset(&ra, 0, sizeof ra);
            ra.B = blocks + L.prep.blk[0].out_off;
            // one-digit row blocks E_w, w in R
            for (size_t rk = 0; rk < vp.R.size(); rk++) {
                int w = vp.R[rk];
                cb = (uint32_t)contrib.size();
                for (int e : vp.edges)
                    if (other_of(e) == w) edge_contrib(e, plan_digit(vp, w));
                for (const auto &t : vp.terms)
                    if (t.dig.size() == 1 && t.dig[0] == w) table_contrib(t);
                if (contrib.size() == cb) continue;
                int b = add_block({}, w, g->K[w], cb);
                ATerm &at = ra.a[ra.na++];
                at.ptr = blocks + L.prep.blk[b].out_off;
                at.sc = g->K[w];
                at.bytes = (uint32_t)(L.prep.blk[b].elems * sizeof(KeyT));
                at.sdR[rk] = 1;
            }
            // lookups touching a row digit with two or more digits: read in the kernel
            for (const auto &t : vp.terms) {
                if (t.dig.size() < 2) continue;
                bool touches = false;
                for (int u : t.dig) touches |= std::count(vp.R.begin(), vp.R.end(), u) > 0;
                if (!touches) continue;
                if (ra.na >= (uint32_t)kMaxATerms) return fail(g, PASE_ERR_INTERNAL, "row terms");
                ATerm &at = ra.a[ra.na++];
                uint32_t sc, sd[kMaxDep];
                lookup_strides(P, i, t.j, sc, sd);
                if (max_index(vp.K, sc, sd, rad, m) >= P.v[t.j].N) bounds_ok = false;
                at.ptr = ws + P.off_T + P.v[t.j].T_off;
                at.sc = sc;
                at.bytes = (uint32_t)(P.v[t.j].N * 8);
                // plan digits: z (if there is a column digit), then O, then R
                const size_t zoff = vp.z >= 0 ? 1 : 0;
                for (size_t k = 0; k < vp.O.size(); k++) at.sdO[k] = sd[zoff + k];
                for (size_t k = 0; k < vp.R.size(); k++) at.sdR[k] = sd[zoff + vp.O.size() + k];
            }
            ra.ldz = vp.ldz;
            ra.Kz = vp.z >= 0 ? g->K[vp.z] : 1;
            ra.K = vp.K;
            ra.bits = vp.bits;
            ra.MO = (uint32_t)vp.MO;
            ra.MR = (uint32_t)vp.MR;
            ra.tiles_per_o = (uint32_t)((vp.MR + 64 * vp.TM - 1) / (64 * vp.TM));
            ra.nchunks = vp.nchunks;
            ra.nsplit = vp.nsplit;
            ra.cper = vp.cper;
            ra.nO = (uint32_t)vp.O.size();
            ra.nR = (uint32_t)vp.R.size();
            for (size_t k = 0; k < vp.O.size(); k++) ra.radO[k] = g->K[vp.O[k]];
            for (size_t k = 0; k < vp.R.size(); k++) ra.radR[k] = g->K[vp.R[k]];
            ra.T = ws + P.off_T + vp.T_off;
            ra.A = (uint16_t *)(ws + P.off_A + vp.A_off);
            ra.partial = ws + P.off_partial + vp.partial_off;
            ra.N = vp.N;
            ra.out_shift = vp.out_shift;
            // a workgroup takes 4 / parts tiles
            ra.parts = vp.parts;
            ra.total_tiles = (uint64_t)vp.nsplit * vp.nchunks * vp.MO * ra.tiles_per_o;
            uint64_t nbk = (ra.total_tiles + 4 / vp.parts - 1) / (4 / vp.parts);
            nbk = (nbk + 7) / 8 * 8;
            if (nbk > 0x7fffffffull) return fail(g, PASE_ERR_TOO_LARGE, "grid too large");
            ra.nblocks_launched = (uint32_t)nbk;
            L.rows = true;
            if (vp.nsplit > 1 || vp.fused_from >= 0) {
                L.red.nblk = grid_for(vp.N);
                L.red.partial = vp.fused_from >= 0 ? (void *)(ws + P.off_fused + vp.fkeys_off) : ra.partial;
                L.red.T = ra.T;
                L.red.A = ra.A;
                L.red.N = vp.N;
                L.red.nsplit = vp.nsplit;
                L.red.bits = vp.bits;
                L.red.out_shift = vp.out_shift;
            }
            if (vp.fused_from >= 0) {
                // the producer's epilogue forms this vertex's keys; its own fill
                // is the reduction of those keys (its row descriptor stays for
                // the producer to copy the row terms from)
                L.rows = false;
                L.fused = true;
                if (vp.nsplit != 1) return fail(g, PASE_ERR_INTERNAL, "fused minimum split over c");
            }
        } else {
            GenericArgs &ga = L.ga;
            std::memset(&ga, 0, sizeof ga);
            uint32_t cb = (uint32_t)contrib.size();
            layer_contrib();
            for (const auto &t : vp.terms)
                if (t.dig.empty()) table_contrib(t);
            int b0 = add_block({}, -1, 1, cb);
            GTerm &g0 = ga.t[ga.nt++];
            g0.ptr = blocks + L.prep.blk[b0].out_off;
            g0.sc = 1;
            for (int w : vp.D) {
                cb = (uint32_t)contrib.size();
                for (int e : vp.edges)
                    if (other_of(e) == w) edge_contrib(e, plan_digit(vp, w));
                for (const auto &t : vp.terms)
                    if (t.dig.size() == 1 && t.dig[0] == w) table_contrib(t);
                if (contrib.size() == cb) continue;
                int b = add_block({}, w, g->K[w], cb);
                GTerm &gt = ga.t[ga.nt++];
                gt.ptr = blocks + L.prep.blk[b].out_off;
                gt.sc = g->K[w];
                gt.sd[plan_digit(vp, w)] = 1;
            }
            for (const auto &t : vp.terms) {
                if (t.dig.size() < 2) continue;
                if (ga.nt >= (uint32_t)kMaxGTerms)
                    return fail(g, PASE_ERR_TOO_LARGE, "too many table lookups for one vertex");
                GTerm &gt = ga.t[ga.nt++];
                gt.ptr = ws + P.off_T + P.v[t.j].T_off;
                lookup_strides(P, i, t.j, gt.sc, gt.sd);
                if (max_index(vp.K, gt.sc, gt.sd, rad, m) >= P.v[t.j].N) bounds_ok = false;
            }
            ga.m = (uint32_t)vp.layout.size();
            ga.K = vp.K;
            ga.bits = vp.bits;
            // lanes per entry: enough threads to fill the GPU, at most one wave, at most K
            ga.group_log2 = 0;
            while (ga.group_log2 < 6 && (vp.N << ga.group_log2) < 65536 && (2u << ga.group_log2) <= vp.K)
                ga.group_log2++;
            for (size_t k = 0; k < vp.layout.size(); k++) ga.rad[k] = g->K[vp.layout[k]];
            ga.T = ws + P.off_T + vp.T_off;
            ga.A = (uint16_t *)(ws + P.off_A + vp.A_off);
            ga.N = vp.N;
            ga.out_shift = vp.out_shift;
            ga.nblk = (uint32_t)std::min<uint64_t>(((vp.N << ga.group_log2) + 255) / 256, 65535);
        }
        if (boff > vp.block_elems) return fail(g, PASE_ERR_INTERNAL, "block scratch overflow");
        if (!bounds_ok) return fail(g, PASE_ERR_INTERNAL, "a table lookup would leave its table");
        if (vp.nsplit > 1 && vp.partial_off + (uint64_t)vp.nsplit * vp.N * sizeof(KeyT) > P.partial_bytes)
            return fail(g, PASE_ERR_INTERNAL, "split scratch overflow");
        if (vp.block_off + boff * sizeof(KeyT) > P.block_bytes)
            return fail(g, PASE_ERR_INTERNAL, "block scratch overflow");
    }
    if (contrib.size() > P.contrib_count) return fail(g, PASE_ERR_INTERNAL, "contribution overflow");
    // fused minima: the producer's epilogue gets the reader's row terms other
    // than the producer's own table, and its column block
    for (int i1 = 0; i1 < n; i1++) {
        const int i2 = P.v[i1].fuse_into;
        if (i2 < 0) continue;
        if constexpr (sizeof(KeyT) != 8) {
            return fail(g, PASE_ERR_INTERNAL, "fused minimum with 128-bit keys");
        } else {
            const VPlan &a = P.v[i1], &b = P.v[i2];
            RowsArgs &r1 = out[i1].ra;
            const RowsArgs &r2 = out[i2].ra;
            if (!out[i1].rows || !out[i2].fused || a.MO != 1 || a.R != b.R || b.fused_from != i1)
                return fail(g, PASE_ERR_INTERNAL, "fused minimum plan");
            const void *Tp = ws + P.off_T + a.T_off;
            int own = 0;
            r1.fz_na = 0;
            for (uint32_t t = 0; t < r2.na; t++) {
                if (r2.a[t].ptr == Tp) {
                    // the reader's lookup of T_i1 must address it as the producer
                    // writes it: [z][r], z stride MR, row strides those of T_i1
                    bool same = r2.a[t].sc == a.MR;
                    for (size_t k = 0; k < a.R.size(); k++) same &= r2.a[t].sdR[k] == a.stride[1 + k];
                    if (!same) return fail(g, PASE_ERR_INTERNAL, "fused minimum lookup layout");
                    own++;
                    continue;
                }
                r1.fz_a[r1.fz_na++] = r2.a[t];
            }
            if (own != 1) return fail(g, PASE_ERR_INTERNAL, "fused minimum lookup");
            r1.fz_keys = ws + P.off_fused + b.fkeys_off;
            r1.fz_B = r2.B;
            r1.fz_ldz = r2.ldz;
            if (r1.Kz != b.K || r2.MR != a.MR) return fail(g, PASE_ERR_INTERNAL, "fused minimum shape");
            // nothing else reads T_i1 unless the tables are kept for queries
            if (!g->keep_tables) r1.T = nullptr;
        }
    }
    return PASE_OK;
}


template pase_status build_launches<double>(pase_graph_t, char *, std::vector<Launch<double>> &,
                                            std::vector<Contrib> &);
template pase_status build_launches<uint64_t>(pase_graph_t, char *, std::vector<Launch<uint64_t>> &,
                                              std::vector<Contrib> &);
template pase_status build_launches<unsigned __int128>(pase_graph_t, char *,
                                                       std::vector<Launch<unsigned __int128>> &,
                                                       std::vector<Contrib> &);

// ------------------------------------------------------------------ constant image and batches
template <typename KeyT>
pase_status build_image(pase_graph_t g, char *ws, char *img, SearchImage &si, bool allow_streams) {
    const Plan &P = g->plan;
    const int n = (int)P.v.size();
    const size_t nv = g->V.size(), ne = g->E.size();
    std::vector<Launch<KeyT>> launches;
    std::vector<Contrib> contrib;
    pase_status st = build_launches<KeyT>(g, ws, launches, contrib);
    if (st != PASE_OK) return st;
    si = SearchImage();
    // two streams only where both have work after the leaves: crossing from one
    // to the other and back costs 10-15 us each time (a search whose lane 1
    // holds level 0 alone: 402 -> 370 us on the Inception graph)
    si.planned_lanes = allow_streams && P.resident && (g->schedule == kSchedBulk || g->schedule == kSchedSplit);
    bool used[kLanes] = {false, false};
    for (const VPlan &vp : P.v) used[vp.lane] |= vp.lane == 0 || vp.slot >= kSplitBatchedLevels;
    si.lanes = si.planned_lanes && used[0] && used[1];
    si.hoist = allow_streams && !si.planned_lanes && P.hoisted > 0;
    si.lane_hoist = si.planned_lanes && P.hoisted > 0;
    // every piece of the image is checked against the end of its region first
    auto region = [&](uint64_t off, uint64_t bytes, uint64_t end, const char *what) {
        return off + bytes <= end && end <= P.off_cfg ? PASE_OK
                                                     : fail(g, PASE_ERR_INTERNAL, std::string("image region: ") + what);
    };

    // the layer costs, their device bytes and the split signatures
    // [off_L, off_ovedge) are written by k_cost_tables on the device: unless
    // the caller overrode the costs, that range is not cleared here, and it is
    // left out of the upload once it is large enough to pay for a second copy
    // call (what the one copy then carries there is overwritten on the device)
    si.upload_costs = g->overridden || P.off_ovedge - P.off_L < (256u << 10);
    if (g->overridden) {
        std::memset(img, 0, P.off_cfg);
    } else {
        std::memset(img, 0, P.off_L);
        std::memset(img + P.off_ovedge, 0, P.off_cfg - P.off_ovedge);
    }
    // one row set per dimension count, shared by the vertices with that count
    uint64_t row_off[kMaxDims + 1] = {0}, off = 0;
    for (size_t d = 0; d < g->ex_rows.size() && d <= (size_t)kMaxDims; d++) {
        row_off[d] = off;
        if (!g->ex_rows[d].empty()) {
            if ((st = region(P.off_ex + off, g->ex_rows[d].size(), P.off_vert, "split rows")) != PASE_OK) return st;
            std::memcpy(img + P.off_ex + off, g->ex_rows[d].data(), g->ex_rows[d].size());
        }
        off += g->ex_rows[d].size();
    }
    std::vector<DevVertex> dvs(nv);
    uint64_t loff = 0;
    for (size_t v = 0; v < nv; v++) {
        DevVertex &x = dvs[v];
        std::memset(&x, 0, sizeof x);
        x.ex_off = row_off[g->V[v].ndims];
        x.L_off = loff;
        x.flops = g->flops[v];
        x.keep_n = g->keep_n[v];
        x.K = g->K[v];
        x.ndims = g->V[v].ndims;
        x.reduce_mask = g->V[v].reduce_mask;
        x.factors = g->factors ? 1 : 0;
        x.bits = P.v[P.pos[v]].bits;
        x.weight_n = g->weight_n[v];
        x.weight_mask = g->V[v].weight_mask;
        if (g->halo) {
            x.input_mask = g->V[v].input_mask;
            for (uint32_t k = 0; k < kMaxDims; k++) {
                x.halo_w[k] = g->V[v].halo[k];
                x.halo_n[k] = g->halo_n[v][k];
                if (x.halo_w[k]) x.halo_mask |= 1u << k;
            }
        }
        loff += g->K[v];
    }
    si.nL = loff;
    if ((st = region(P.off_vert, nv * sizeof(DevVertex), P.off_edge, "vertices")) != PASE_OK) return st;
    std::memcpy(img + P.off_vert, dvs.data(), nv * sizeof(DevVertex));
    std::vector<DevEdge> des(ne);
    uint64_t sig_off = 0;
    for (size_t e = 0; e < ne; e++) {
        DevEdge &x = des[e];
        std::memset(&x, 0, sizeof x);
        x.src = g->E[e].src;
        x.dst = g->E[e].dst;
        x.rank = g->E[e].rank;
        x.factors = g->factors ? 1 : 0;
        for (uint32_t k = 0; k < kMaxDims; k++) {
            x.sdim[k] = (int8_t)(k < x.rank ? g->E[e].src_dim[k] : -1);
            x.ddim[k] = (int8_t)(k < x.rank ? g->E[e].dst_dim[k] : -1);
        }
        x.elems = g->E[e].elems;
        // its cost enters the keys of the end that comes first in the sequence
        x.bits = P.v[std::min(P.pos[x.src], P.pos[x.dst])].bits;
        x.sig_off = sig_off;
        x.mat_off = g->volume ? g->mat_off[e] : 0;
        x.row0 = g->volume ? g->mat_row0[e] : 0;
        sig_off += (uint64_t)g->K[x.src] + g->K[x.dst];
    }
    if (ne) {
        if ((st = region(P.off_edge, ne * sizeof(DevEdge), P.off_L, "edges")) != PASE_OK) return st;
        std::memcpy(img + P.off_edge, des.data(), ne * sizeof(DevEdge));
    }
    if (g->overridden) {
        if ((st = region(P.off_L, g->ov_layer.size() * 8, P.off_lsum, "layer costs")) != PASE_OK) return st;
        std::memcpy(img + P.off_L, g->ov_layer.data(), g->ov_layer.size() * 8);
        if (!g->ov_edge.empty()) {
            if ((st = region(P.off_ovedge, g->ov_edge.size() * 8, P.off_contrib, "edge costs")) != PASE_OK) return st;
            std::memcpy(img + P.off_ovedge, g->ov_edge.data(), g->ov_edge.size() * 8);
        }
    }
    if ((st = region(P.off_contrib, contrib.size() * sizeof(Contrib), P.off_bt, "contributions")) != PASE_OK) return st;
    if (!contrib.empty()) std::memcpy(img + P.off_contrib, contrib.data(), contrib.size() * sizeof(Contrib));
    std::vector<BacktrackDesc> bt(n);
    uint32_t nlev = 0;
    for (int i = n - 1; i >= 0; i--) {
        const VPlan &vp = P.v[i];
        BacktrackDesc &b = bt[i];
        std::memset(&b, 0, sizeof b);
        b.A = (const uint16_t *)(ws + P.off_A + vp.A_off);
        b.vi = (uint32_t)vp.vi;
        b.K = vp.K;
        b.pos = (uint32_t)i;
        // a vertex whose table is not formed: one evaluation of its terms
        if (vp.absorbed >= 0 && !g->keep_tables)
            b.lazy = (const ClassArgs *)(ws + P.off_desc[kDescClass]) + vp.desc[kDescClass];
        b.m = (uint32_t)vp.layout.size();
        for (size_t k = 0; k < vp.layout.size(); k++) {
            b.dig[k] = (uint32_t)vp.layout[k];
            b.stride[k] = vp.stride[k];
        }
        // the configuration of v_i needs those of D(i), all later in the order
        for (int u : vp.D) b.level = std::max(b.level, bt[P.pos[u]].level + 1);
        nlev = std::max(nlev, b.level + 1);
    }
    si.nlev = nlev;
    if ((st = region(P.off_bt, n * sizeof(BacktrackDesc), P.off_desc[0], "back-substitution")) != PASE_OK) return st;
    std::memcpy(img + P.off_bt, bt.data(), n * sizeof(BacktrackDesc));

    // ---- kernel descriptors, by kind
    for (int k = 0; k < kDescKinds; k++)
        if ((st = region(P.off_desc[k], P.ndesc[k] * kDescBytes[k], k + 1 < kDescKinds ? P.off_desc[k + 1] : P.off_batch,
                         "descriptors")) != PASE_OK)
            return st;
    bool no_desc = false;   // a descriptor index past those of its kind
    auto has_desc = [&](int i, DescKind k) {
        no_desc |= P.v[i].desc[k] >= P.ndesc[k];
        return P.v[i].desc[k] < P.ndesc[k];
    };
    auto put = [&](int i, DescKind k, const auto &src) {
        if (P.v[i].desc[k] == ~0u) return;   // the vertex has none of this kind
        no_desc |= sizeof src != kDescBytes[k];
        if (has_desc(i, k)) std::memcpy(img + P.off_desc[k] + P.v[i].desc[k] * kDescBytes[k], &src, kDescBytes[k]);
    };
    for (int i = 0; i < n; i++) {
        const Launch<KeyT> &L = launches[i];
        put(i, kDescPrep, L.prep);
        put(i, kDescRows, L.ra);
        put(i, kDescGeneric, L.ga);
        put(i, kDescReduce, L.red);
        put(i, kDescDirect, L.da);
        put(i, kDescClass, L.ca);
        put(i, kDescJoint, L.ja);
        put(i, kDescExch, L.xa);
        if (P.v[i].absorbed >= 0 && !g->keep_tables) has_desc(i, kDescClass);   // (read by the back-substitution)
    }
    if (no_desc) return fail(g, PASE_ERR_INTERNAL, "a descriptor past those of its kind");
    RowsArgs *hr = (RowsArgs *)(img + P.off_desc[kDescRows]);
    if (!P.ctabs.empty()) {
        if ((st = region(P.off_ctdesc, P.ctabs.size() * sizeof(DevClassTab), P.off_jtdesc, "class tables")) != PASE_OK) return st;
        if ((st = region(P.off_jtdesc, P.jtabs.size() * sizeof(DevJointTab), P.off_zero, "joint tables")) != PASE_OK) return st;
        if (!P.jtabs.empty()) std::memcpy(img + P.off_jtdesc, P.jtabs.data(), P.jtabs.size() * sizeof(DevJointTab));
        DevClassTab *ht = (DevClassTab *)(img + P.off_ctdesc);
        for (size_t k = 0; k < P.ctabs.size(); k++) {
            ht[k] = P.ctabs[k];
            ht[k].ex_u = row_off[ht[k].ndu];
            ht[k].ex_z = row_off[ht[k].ndz];
        }
    }

    // ---- batches: per launch group, one prep launch, one fill launch per
    // kernel variant and one split-reduction launch
    BatchEntry *hbe = (BatchEntry *)(img + P.off_batch);
    const uint64_t be_cap = (P.off_ctdesc - P.off_batch) / sizeof(BatchEntry);
    uint32_t nbe = 0;
    // launch groups in enqueue order: the slots (levels, or positions); with
    // lanes, each slot's vertices of lane 0, then those of lane 1
    const int nl = si.lanes ? kLanes : 1;
    si.groups.assign((size_t)P.nslots * nl, {});
    si.group_lane.assign(si.groups.size(), 0);
    for (int i = 0; i < n; i++) si.groups[(size_t)P.v[i].slot * nl + (si.lanes ? P.v[i].lane : 0)].push_back(i);
    for (size_t k = 0; k < si.groups.size(); k++) si.group_lane[k] = (int)(k % nl);
    int cur_lane = 0, cur_group = 0;
    bool be_overflow = false;
    auto add_batch = [&](Batch::Kind kind, uint32_t variant, const std::vector<int> &members,
                         uint32_t (*nblk)(const Launch<KeyT> &)) {
        if (members.empty()) return;
        Batch b{kind, cur_lane, cur_group, variant, nbe, 0, 0};
        static const DescKind kind_of[] = {kDescPrep, kDescRows, kDescGeneric, kDescReduce,
                                           kDescDirect, kDescClass, kDescJoint, kDescJoint, kDescExch, kDescExch};
        b.idx0 = P.v[members[0]].desc[kind_of[kind]];
        for (int i : members) {
            if (kind == Batch::kJoint) b.lds = std::max(b.lds, launches[i].ja.lds);
            if (kind == Batch::kHalf) b.lds = std::max(b.lds, launches[i].ja.hlds);
            if (kind == Batch::kExchHalf) b.lds = std::max(b.lds, launches[i].xa.lds);
            if (kind == Batch::kClass) b.lds = std::max(b.lds, launches[i].ca.lds);
            if (nbe >= be_cap) { be_overflow = true; return; }
            hbe[nbe].pos = (uint32_t)i;
            hbe[nbe].idx = P.v[i].desc[kind_of[kind]];
            if (!has_desc(i, kind_of[kind])) return;
            hbe[nbe].first = b.blocks;
            hbe[nbe].prio = si.lanes && P.v[i].lane == 0 ? 1u : 0u;
            hbe[nbe].kind = 0;
            b.blocks += nblk(launches[i]);
            nbe++;
            b.nentries++;
        }
        si.batches.push_back(b);
    };
    // per-group scratch, reused across groups (cleared, capacity kept)
    std::vector<int> prepped, direct, cls, joint, half, exch, exch_half, grp;
    std::vector<std::pair<uint32_t, int>> rows, gens, reds;
    std::map<uint32_t, int> shape_dom;   // TZ * 4 + TM -> largest vertex of the group
    constexpr bool kF64 = std::is_same<KeyT, double>::value;
    // hoisted preps: a side batch after the group of the slot whose tables
    // they read last (before group 0 when they read none); each vertex's group
    // waits for its side batch
    std::vector<std::vector<int>> hoist_after(si.groups.size() + 1);   // [slot + 1] -> positions
    si.group_waits.assign(si.groups.size(), {});
    if (si.hoist)
        for (int i = 0; i < n; i++)
            if (P.v[i].prep_after >= -1 && P.v[i].joint < 0) hoist_after[(size_t)(P.v[i].prep_after + 1)].push_back(i);
    // with lanes: a hoisted prep is a prep batch of its own at the end of the
    // group (prep_after, lane of the tables it reads)
    std::vector<std::vector<int>> lane_hoist_at(si.groups.size());   // group -> positions
    if (si.lane_hoist)
        for (int i = 0; i < n; i++)
            if (P.v[i].prep_after >= 0 && P.v[i].joint < 0)
                lane_hoist_at[(size_t)P.v[i].prep_after * nl + (si.lanes ? P.v[i].prep_lane : 0)].push_back(i);
    const bool hoisting = si.hoist || si.lane_hoist;
    auto add_side = [&](size_t k) {
        if (hoist_after[k].empty()) return;
        const int bi = (int)si.batches.size();
        add_batch(Batch::kPrep, 0, hoist_after[k], [](const Launch<KeyT> &L) { return L.prep.nwg; });
        if ((int)si.batches.size() == bi + 1) si.batches.back().side = true;
        for (int i : hoist_after[k]) si.group_waits[(size_t)P.v[i].slot].push_back(bi);
    };
    add_side(0);
    for (size_t sl = 0; sl < si.groups.size(); sl++) {
        const auto &mem = si.groups[sl];
        cur_lane = si.group_lane[sl];
        cur_group = (int)sl;
        prepped.clear();
        direct.clear();
        cls.clear();
        joint.clear();
        half.clear();
        exch.clear();
        exch_half.clear();
        // a fused minimum's blocks are built with its producer's, before the
        // producer's fill reads them; its own fill is a reduction (below)
        std::vector<int> fills;   // members with a prep here or hoisted: rows / generic fills
        for (int i : mem) {
            // (the half fill of a joint fill carries that fill's position)
            if (P.v[i].absorbed >= 0) {
                const VPlan &by = P.v[P.v[i].absorbed];
                if (by.jearly) (by.exch ? exch_half : half).push_back(P.v[i].absorbed);
                if (!g->keep_tables) continue;   // no table of its own
            }
            if (launches[i].joint) {
                (P.v[i].exch ? exch : joint).push_back(i);
                if (!P.v[i].jearly) (P.v[i].exch ? exch_half : half).push_back(i);
                continue;
            }
            if (launches[i].cls) cls.push_back(i);
            else if (launches[i].direct) direct.push_back(i);
            else if (!launches[i].fused) (hoisting && P.v[i].prep_after >= -1 ? fills : prepped).push_back(i);
            if (P.v[i].fuse_into >= 0) prepped.push_back(P.v[i].fuse_into);
        }
        add_batch(Batch::kDirect, 0, direct, [](const Launch<KeyT> &L) { return L.da.nblk; });
        // class fills: one launch for the vertices of at most two edges and two
        // lookups, one for the others
        for (uint32_t many = 0; many < 2; many++) {
            uint32_t threads = 256;
            grp.clear();
            for (int i : cls)
                if ((launches[i].ca.ne > 2 || launches[i].ca.nt > 2) == (many == 1)) {
                    grp.push_back(i);
                    threads = std::max(threads, P.v[i].threads);
                }
            add_batch(Batch::kClass, threads + many, grp, [](const Launch<KeyT> &L) { return L.ca.nblk; });
        }
        add_batch(Batch::kPrep, 0, prepped, [](const Launch<KeyT> &L) { return L.prep.nwg; });
        uint32_t half_threads = 64;
        for (int i : half) half_threads = std::max(half_threads, std::min<uint32_t>(512, launches[i].ja.threads));
        add_batch(Batch::kHalf, half_threads, half, [](const Launch<KeyT> &L) { return L.ja.hblk; });
        add_batch(Batch::kExchHalf, 0, exch_half, [](const Launch<KeyT> &L) { return L.xa.Kj; });
        add_batch(Batch::kExch, 0, exch, [](const Launch<KeyT> &L) { return L.xa.nblk; });
        // joint fills: one launch for one configuration per thread, one for two
        for (uint32_t two = 0; two < 2; two++) {
            uint32_t threads = 64;
            grp.clear();
            for (int i : joint) {
                const JointArgs &ja = launches[i].ja;
                const uint32_t most = std::max(std::max(ja.s[0].K, ja.s[1].K), ja.Ky);
                if ((most > ja.threads) == (two == 1)) {
                    grp.push_back(i);
                    threads = std::max(threads, ja.threads);
                }
            }
            add_batch(Batch::kJoint, threads + two, grp, [](const Launch<KeyT> &L) { return L.ja.nblk; });
        }
        prepped.insert(prepped.end(), fills.begin(), fills.end());
        rows.clear();
        gens.clear();
        reds.clear();
        // fp64 keys: the row-term count is a kernel template parameter; a
        // small vertex with fewer row terms than the largest vertex of its tile
        // shape in this group gets zero terms appended (each lane adds the
        // zero key once per c) and joins that vertex's launch
        shape_dom.clear();
        for (int i : prepped)
            if (launches[i].rows && !launches[i].fused && kF64) {
                auto it = shape_dom.find(P.v[i].TZ * 4 + P.v[i].TM);
                if (it == shape_dom.end()) shape_dom[P.v[i].TZ * 4 + P.v[i].TM] = i;
                else if (P.v[i].est_us > P.v[it->second].est_us) it->second = i;
            }
        for (int i : prepped) {
            const Launch<KeyT> &L = launches[i];
            if (L.fused) continue;
            if (L.rows) {
                uint32_t na = kF64 ? std::min<uint32_t>(L.ra.na, 4) : 7;
                if (kF64) {
                    const int d = shape_dom[P.v[i].TZ * 4 + P.v[i].TM];
                    const uint32_t nd = std::min<uint32_t>(launches[d].ra.na, 4);
                    if (d != i && na < nd && P.v[i].est_us <= 0.5 * P.v[d].est_us && has_desc(i, kDescRows)) {
                        RowsArgs &ra = hr[P.v[i].desc[kDescRows]];
                        for (uint32_t t = na; t < nd; t++) {
                            std::memset(&ra.a[t], 0, sizeof ra.a[t]);
                            ra.a[t].ptr = ws + P.off_zero;
                            ra.a[t].bytes = 8;
                        }
                        na = nd;
                    }
                }
                rows.push_back({(P.v[i].TZ * 4 + P.v[i].TM) * 8 + na, i});
                if (P.v[i].nsplit > 1) reds.push_back({0, i});
            } else {
                gens.push_back({L.ga.nt <= 6 ? L.ga.nt : 0, i});
            }
        }
        auto by_variant = [](const std::pair<uint32_t, int> &a, const std::pair<uint32_t, int> &b) {
            return a.first < b.first;
        };
        std::stable_sort(rows.begin(), rows.end(), by_variant);
        std::stable_sort(gens.begin(), gens.end(), by_variant);
        // two-term generic fills of the group ride along in its largest row
        // launch (64-bit keys) instead of a generic launch of their own
        std::vector<int> ride;
        uint32_t ride_variant = ~0u;
        if constexpr (sizeof(KeyT) == 8) {
            uint64_t best = 0;
            for (size_t k = 0; k < rows.size();) {
                size_t k2 = k;
                uint64_t blocks = 0;
                for (; k2 < rows.size() && rows[k2].first == rows[k].first; k2++)
                    blocks += launches[rows[k2].second].ra.nblocks_launched;
                if (ride_variant == ~0u || blocks > best) { best = blocks; ride_variant = rows[k].first; }
                k = k2;
            }
            if (ride_variant != ~0u) {
                std::vector<std::pair<uint32_t, int>> keep;
                for (const auto &x : gens) {
                    if (launches[x.second].ga.nt == 2) ride.push_back(x.second);
                    else keep.push_back(x);
                }
                gens.swap(keep);
            }
        }
        for (size_t k = 0; k < rows.size();) {
            grp.clear();
            size_t k2 = k;
            for (; k2 < rows.size() && rows[k2].first == rows[k].first; k2++) grp.push_back(rows[k2].second);
            add_batch(Batch::kRows, rows[k].first, grp, [](const Launch<KeyT> &L) { return L.ra.nblocks_launched; });
            if (rows[k].first == ride_variant && !si.batches.empty()) {
                Batch &b = si.batches.back();
                for (int i : ride) {
                    if (nbe >= be_cap) { be_overflow = true; break; }
                    hbe[nbe].pos = (uint32_t)i;
                    hbe[nbe].idx = P.v[i].desc[kDescGeneric];
                    if (!has_desc(i, kDescGeneric)) break;
                    hbe[nbe].first = b.blocks;
                    hbe[nbe].prio = si.lanes && P.v[i].lane == 0 ? 1u : 0u;
                    hbe[nbe].kind = kEntryGeneric2;
                    b.blocks += launches[i].ga.nblk;
                    nbe++;
                    b.nentries++;
                }
            }
            k = k2;
        }
        for (size_t k = 0; k < gens.size();) {
            grp.clear();
            size_t k2 = k;
            for (; k2 < gens.size() && gens[k2].first == gens[k].first; k2++) grp.push_back(gens[k2].second);
            add_batch(Batch::kGeneric, gens[k].first, grp, [](const Launch<KeyT> &L) { return L.ga.nblk; });
            k = k2;
        }
        for (int i : mem)
            if (launches[i].fused) reds.push_back({0, i});
        grp.clear();
        for (auto &x : reds) grp.push_back(x.second);
        add_batch(Batch::kReduce, 0, grp, [](const Launch<KeyT> &L) { return L.red.nblk; });
        add_batch(Batch::kPrep, 0, lane_hoist_at[sl], [](const Launch<KeyT> &L) { return L.prep.nwg; });
        if (no_desc) return fail(g, PASE_ERR_INTERNAL, "a launch without a descriptor");
        if (be_overflow) return fail(g, PASE_ERR_INTERNAL, "batch table overflow");
        add_side(sl + 1);
    }
    for (const Batch &b : si.batches)
        if (b.blocks == 0 || b.blocks > 0x7fffffffu) return fail(g, PASE_ERR_TOO_LARGE, "launch grid size");
    return PASE_OK;
}

template pase_status build_image<double>(pase_graph_t, char *, char *, SearchImage &, bool);
template pase_status build_image<uint64_t>(pase_graph_t, char *, char *, SearchImage &, bool);
template pase_status build_image<unsigned __int128>(pase_graph_t, char *, char *, SearchImage &, bool);

pase_status plan_check(pase_graph_t g, uint64_t *image_bytes) {
    // descriptors only hold device addresses: any base will do, nothing is
    // read through it; the image buffer is exactly the constant region, so a
    // write past it is a heap overflow (and a sanitizer build reports it)
    char *fake_ws = (char *)(uintptr_t)(1ull << 40);
    const uint64_t bytes = g->plan.off_cfg;
    std::vector<char> img(bytes);
    SearchImage si;
    pase_status st = g->plan_key_type == 0   ? build_image<double>(g, fake_ws, img.data(), si)
                     : g->plan_key_type == 1 ? build_image<uint64_t>(g, fake_ws, img.data(), si)
                                             : build_image<unsigned __int128>(g, fake_ws, img.data(), si);
    if (st != PASE_OK) return st;
    // every vertex appears in exactly one fill batch (direct, row or generic)
    std::vector<int> fills(g->plan.v.size(), 0);
    const BatchEntry *be = (const BatchEntry *)(img.data() + g->plan.off_batch);
    std::vector<int> prep_batch(g->plan.v.size(), -1), fill_batch(g->plan.v.size(), -1), half_batch(g->plan.v.size(), -1);
    for (size_t bi = 0; bi < si.batches.size(); bi++) {
        const Batch &b = si.batches[bi];
        for (uint32_t k = 0; k < b.nentries; k++) {
            const uint32_t pos = be[b.entry0 + k].pos;
            if (pos >= fills.size()) return fail(g, PASE_ERR_INTERNAL, "batch entry out of range");
            const bool fused = g->plan.v[pos].fused_from >= 0;
            if (b.kind == Batch::kRows || b.kind == Batch::kGeneric || b.kind == Batch::kDirect ||
                b.kind == Batch::kClass || b.kind == Batch::kJoint || b.kind == Batch::kExch ||
                (b.kind == Batch::kReduce && fused)) {
                fills[pos]++;
                fill_batch[pos] = (int)bi;
            }
            if (b.kind == Batch::kPrep) prep_batch[pos] = (int)bi;
            if (b.kind == Batch::kHalf || b.kind == Batch::kExchHalf) half_batch[pos] = (int)bi;
        }
    }
    // every vertex with blocks has them built before its fill; a hoisted
    // prep's side batch comes after the fills of the slot it waits for and is
    // waited for by the vertex's group
    for (size_t i = 0; i < g->plan.v.size(); i++) {
        const VPlan &vp = g->plan.v[i];
        if (vp.kernel == kDirect || vp.classes || vp.joint >= 0 || vp.fused_from >= 0 || fill_batch[i] < 0) continue;
        if (prep_batch[i] < 0 || prep_batch[i] > fill_batch[i])
            return fail(g, PASE_ERR_INTERNAL, "a prep does not precede its fill");
        if (si.hoist && vp.prep_after >= -1) {
            const Batch &b = si.batches[prep_batch[i]];
            const auto &w = si.group_waits[(size_t)vp.slot];
            if (!b.side || std::find(w.begin(), w.end(), prep_batch[i]) == w.end())
                return fail(g, PASE_ERR_INTERNAL, "a hoisted prep is not waited for");
            for (size_t k = 0; k < (size_t)prep_batch[i]; k++)
                if (si.batches[k].group > vp.prep_after && !si.batches[k].side)
                    return fail(g, PASE_ERR_INTERNAL, "a hoisted prep runs after a later slot");
            for (size_t k = prep_batch[i] + 1; k < si.batches.size(); k++)
                if (si.batches[k].group <= vp.prep_after && !si.batches[k].side)
                    return fail(g, PASE_ERR_INTERNAL, "a hoisted prep runs before the tables it reads");
        }
        // with lanes: at the end of group (prep_after, prep_lane), after the
        // fills of that lane's tables up to that slot (the ones its blocks
        // read among them); on another lane than the vertex's, the vertex
        // reads a table of the prep's lane at that slot or later, so its group
        // waits for that lane past the prep
        if (si.lane_hoist && vp.prep_after >= 0) {
            const Batch &b = si.batches[prep_batch[i]];
            const int lane = si.lanes ? vp.prep_lane : 0, nl = si.lanes ? kLanes : 1;
            if (b.lane != lane || b.group != vp.prep_after * nl + lane)
                return fail(g, PASE_ERR_INTERNAL, "a hoisted prep is not on its lane");
            bool waited = !si.lanes || vp.prep_lane == vp.lane;
            bool early = false;
            for_reads(g->plan, vp, [&](int j) {
                const VPlan &pj = g->plan.v[j];
                early |= pj.slot <= vp.prep_after && pj.lane == vp.prep_lane && fill_batch[j] > prep_batch[i];
                waited |= pj.lane == vp.prep_lane && pj.slot >= vp.prep_after;
            });
            if (early) return fail(g, PASE_ERR_INTERNAL, "a hoisted prep runs before the tables it reads");
            if (!waited) return fail(g, PASE_ERR_INTERNAL, "a hoisted prep on another lane is not waited for");
        }
    }
    // every table a launch reads is filled before it, in an earlier slot (a
    // joint fill reads the other vertex's half fill, that one its lookups)
    for (size_t i = 0; i < g->plan.v.size(); i++) {
        const VPlan &vp = g->plan.v[i];
        if (fill_batch[i] < 0) continue;
        if (vp.joint >= 0 && (half_batch[i] < 0 || half_batch[i] >= fill_batch[i]))
            return fail(g, PASE_ERR_INTERNAL, "a half fill does not precede its joint fill");
        bool early = false;
        for_reads(g->plan, vp, [&](int j) {
            early |= j != vp.joint && (fill_batch[j] < 0 || fill_batch[j] >= fill_batch[i] || g->plan.v[j].slot >= vp.slot);
        });
        if (early) return fail(g, PASE_ERR_INTERNAL, "a table is read before it is filled");
        if (vp.joint >= 0)
            for (const auto &t : g->plan.v[vp.joint].terms)
                if (fill_batch[t.j] < 0 || fill_batch[t.j] >= half_batch[i])
                    return fail(g, PASE_ERR_INTERNAL, "a half fill reads a table before it is filled");
    }
    // a fused minimum: its blocks are built before its producer's fill, and its
    // reduction comes after that fill
    for (size_t i = 0; i < g->plan.v.size(); i++) {
        const int j = g->plan.v[i].fused_from;
        if (j < 0) continue;
        if (prep_batch[i] < 0 || fill_batch[j] < 0 || prep_batch[i] > fill_batch[j] || fill_batch[i] < fill_batch[j])
            return fail(g, PASE_ERR_INTERNAL, "fused minimum out of order");
    }
    for (size_t i = 0; i < fills.size(); i++)
        if (fills[i] != (g->plan.v[i].absorbed >= 0 && !g->keep_tables ? 0 : 1)) return fail(g, PASE_ERR_INTERNAL, "a vertex is not filled exactly once");
    *image_bytes = bytes;
    return PASE_OK;
}

}  // namespace pase
