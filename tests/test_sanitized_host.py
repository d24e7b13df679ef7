"""The host code of libpase (planner, launch planning, constant-region image)
under AddressSanitizer and UBSan: a host-only build with a stub device
runtime runs the whole host test suite in a child process with the ASan
runtime preloaded; any report aborts the child and fails this test."""
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def san_lib():
    if not shutil.which(os.environ.get("CXX", "g++")):
        pytest.skip("no host C++ compiler")
    from paper_2407_04001_amd import build
    return build.build_host_sanitized()


def test_host_suite_under_address_and_undefined_behaviour_sanitizers(san_lib):
    cxx = shutil.which(os.environ.get("CXX", "g++"))
    lib = san_lib
    asan = subprocess.run([cxx, "-print-file-name=libasan.so"], capture_output=True, text=True).stdout.strip()
    assert os.path.isabs(asan) and os.path.exists(asan), asan
    env = dict(os.environ, LD_PRELOAD=asan,
               ASAN_OPTIONS="detect_leaks=0:abort_on_error=1:halt_on_error=1",
               UBSAN_OPTIONS="halt_on_error=1:print_stacktrace=1")
    cmd = [sys.executable, "-m", "pytest", os.path.join(ROOT, "tests", "test_host.py"), "-q", "-x",
           "-p", "no:cacheprovider", "--pase-lib", lib]
    r = subprocess.run(cmd, cwd=ROOT, env=env, capture_output=True, text=True, timeout=1200)
    tail = (r.stdout + r.stderr)[-4000:]
    assert r.returncode == 0, tail
    assert " passed" in r.stdout, tail


# A chain whose middle vertices take the class fill (or, in the generic kernel
# mode, prep + generic fills); then one vertex's descriptor index, or the number
# of descriptors the memory layout made room for, is put out of step with the
# other, as a planner mistake would.
DESCRIPTORS = r"""
#include <cstdio>
#include <cstring>
#include "internal.h"
using namespace pase;
int main() {
    for (int mode = 0; mode < 2; mode++) {
        pase_vertex_desc v[5];
        pase_edge_desc e[4];
        std::memset(v, 0, sizeof v);
        std::memset(e, 0, sizeof e);
        for (auto &x : v) { x.ndims = 2; x.size[0] = x.size[1] = 64; x.flops_per_point = 2; }
        for (uint32_t k = 0; k < 4; k++) {
            e[k].src = k; e[k].dst = k + 1; e[k].rank = 1; e[k].elems = 64;
        }
        pase_cost_params par{8, 0};
        pase_graph_t g;
        if (pase_graph_create(v, 5, e, 4, &par, &g) != PASE_OK) return 1;
        pase_set_option(g, PASE_OPT_KERNEL, mode);
        if (pase_enumerate_configs(g, 16) != PASE_OK) return 2;
        uint64_t bytes;
        if (pase_plan_check(g, &bytes) != PASE_OK) return 3;
        int kinds = 0;
        for (int k = 0; k < kDescKinds; k++) {
            Plan &P = g->plan;
            if (!P.ndesc[k]) continue;
            kinds++;
            uint32_t *at = nullptr;
            for (auto &vp : P.v)
                if (vp.desc[k] != ~0u) at = &vp.desc[k];
            const uint32_t was = *at, n = P.ndesc[k];
            *at = n;            // one past the last
            if (pase_plan_check(g, &bytes) != PASE_ERR_INTERNAL) return 10 + k;
            *at = was;
            P.ndesc[k] = n - 1; // room for one fewer
            if (pase_plan_check(g, &bytes) != PASE_ERR_INTERNAL) return 20 + k;
            P.ndesc[k] = n + (uint32_t)((P.off_zero - P.off_desc[k]) / kDescBytes[k]) + 1;   // past its region
            if (pase_plan_check(g, &bytes) != PASE_ERR_INTERNAL) return 30 + k;
            P.ndesc[k] = n;
            if (pase_plan_check(g, &bytes) != PASE_OK) return 4;
        }
        if (!kinds) return 5;
        pase_graph_destroy(g);
    }
    std::puts("descriptors ok");
}
"""


# Caller-given costs on a graph planned for the model's own, and back: the
# fills are planned again, the sequence and the dependent sets are not.
OVERRIDE = r"""
#include <cstdio>
#include <cstring>
#include "internal.h"
using namespace pase;
int main() {
    pase_vertex_desc v[6];
    pase_edge_desc e[6];
    std::memset(v, 0, sizeof v);
    std::memset(e, 0, sizeof e);
    for (auto &x : v) { x.ndims = 2; x.size[0] = x.size[1] = 64; x.flops_per_point = 2; }
    for (uint32_t k = 0; k < 6; k++) {
        e[k].src = k < 5 ? k : 0; e[k].dst = k < 5 ? k + 1 : 3; e[k].rank = 1; e[k].elems = 64;
    }
    pase_cost_params par{8, 0};
    pase_graph_t g;
    if (pase_graph_create(v, 6, e, 6, &par, &g) != PASE_OK) return 1;
    if (pase_enumerate_configs(g, 16) != PASE_OK) return 2;
    const auto seq = g->plan.seq;
    const auto D = g->plan.v[1].D;
    const uint32_t fills = g->plan.class_fills;
    std::vector<uint64_t> layer, edge;
    for (uint32_t k : g->K) layer.resize(layer.size() + k, 3);
    for (auto &x : g->E) edge.resize(edge.size() + (size_t)g->K[x.src] * g->K[x.dst], 5);
    g->stats.seq_ms = -7;   // (set whenever the sequence is formed)
    uint64_t bytes;
    for (int turn = 0; turn < 2; turn++) {
        if (pase_override_costs(g, layer.data(), edge.data()) != PASE_OK) return 3;
        if (g->stats.seq_ms != -7) return 4;
        if (g->plan.seq != seq || g->plan.v[1].D != D || g->plan.class_fills) return 5;
        if (pase_plan_check(g, &bytes) != PASE_OK) return 6;
        // the bounds are those of the new costs: one layer cost and up to two edges per vertex, and its lookups
        if (g->plan.qmax[0] != (turn ? 1000u : 3u) + 5 * g->plan.v[0].edges.size()) return 7;
        for (auto &x : layer) x = 1000;
    }
    if (pase_enumerate_configs(g, 16) != PASE_OK || g->plan.class_fills != fills || !fills) return 8;
    pase_graph_destroy(g);
    std::puts("override ok");
}
"""


# Chains of small vertices of 462 configurations, whose class fills need more
# memory than the dense ones: at a memory budget, a lent workspace and the
# static workspace that only the dense fills fit, the search is not refused.
LIMITS = r"""
#include <cstdio>
#include <cstring>
#include "internal.h"
using namespace pase;
static pase_graph_t chain(uint32_t n) {
    std::vector<pase_vertex_desc> v(n);
    std::vector<pase_edge_desc> e(n - 1);
    std::memset(v.data(), 0, n * sizeof v[0]);
    std::memset(e.data(), 0, (n - 1) * sizeof e[0]);
    for (auto &x : v) { x.ndims = 5; for (int k = 0; k < 5; k++) x.size[k] = 64; x.flops_per_point = 2; }
    for (uint32_t k = 0; k + 1 < n; k++) { e[k].src = k; e[k].dst = k + 1; e[k].rank = 1; e[k].elems = 64; }
    pase_cost_params par{8, 0};
    pase_graph_t g = nullptr;
    if (pase_graph_create(v.data(), n, e.data(), n - 1, &par, &g) != PASE_OK) return nullptr;
    return pase_enumerate_configs(g, 64) == PASE_OK ? g : nullptr;
}
static void sizes(uint32_t n, uint64_t &all, uint64_t &dense) {
    pase_graph_t g = chain(n);
    pase_workspace_size(g, &all);
    pase_set_option(g, PASE_OPT_C_SPLITS, 1);   // (a tile knob: the dense fills)
    pase_workspace_size(g, &dense);
    pase_graph_destroy(g);
}
int main() {
    uint64_t all = 0, dense = 0, mc = 0, now = 0, bytes = 0;
    std::vector<uint32_t> cfg(20000);
    sizes(40, all, dense);
    if (all <= dense + 131072) return 1;
    // a memory budget that the structured fills pass
    pase_graph_t g = chain(40);
    if (pase_set_option(g, PASE_OPT_MEMORY_BUDGET, dense + 65536) != PASE_OK) return 2;
    if (pase_workspace_size(g, &now) != PASE_OK || now > dense + 65536 || !g->dense_only || g->plan.class_fills) return 3;
    if (pase_plan_check(g, &bytes) != PASE_OK) return 4;
    if (pase_set_option(g, PASE_OPT_MEMORY_BUDGET, 64ull << 30) != PASE_OK || g->dense_only || !g->plan.class_fills) return 5;
    // a lent workspace (the host-only build stops where the device work would begin)
    void *lent = (void *)(uintptr_t)4096;
    for (int turn = 0; turn < 2; turn++) {
        pase_set_workspace(g, lent, dense + 65536);
        if (pase_find_best_strategy(g, nullptr, &mc, cfg.data()) != PASE_ERR_HIP || !g->dense_only) return 6;
        pase_set_workspace(g, lent, all);
        if (pase_find_best_strategy(g, nullptr, &mc, cfg.data()) != PASE_ERR_HIP || g->dense_only) return 7;
    }
    pase_set_workspace(g, lent, 100000);   // neither fits: refused, and planned as before
    if (pase_find_best_strategy(g, nullptr, &mc, cfg.data()) != PASE_ERR_OUT_OF_MEMORY) return 8;
    if (g->dense_only || pase_workspace_size(g, &now) != PASE_OK || now != all) return 9;
    pase_graph_destroy(g);
    // the static workspace
    uint64_t all2, dense2;
    sizes(80, all2, dense2);
    const uint32_t n = (uint32_t)(40 + (PASE_NOALLOC_WORKSPACE_BYTES - (1u << 20) - dense) / ((dense2 - dense) / 40));
    g = chain(n);
    if (pase_workspace_size(g, &now) != PASE_OK || now <= PASE_NOALLOC_WORKSPACE_BYTES) return 10;
    if (pase_find_best_strategy_noalloc(g, nullptr, &mc, cfg.data()) != PASE_ERR_HIP) return 11;
    if (!g->dense_only || g->plan.total > PASE_NOALLOC_WORKSPACE_BYTES) return 12;
    if (pase_find_best_strategy(g, nullptr, &mc, cfg.data()) != PASE_ERR_HIP || g->dense_only) return 13;
    pase_graph_destroy(g);
    std::puts("limits ok");
}
"""


def host_program(source, lib, tmp_path, expect):
    src = tmp_path / "program.cpp"
    src.write_text(source)
    exe = str(tmp_path / "program")
    subprocess.run([os.environ.get("CXX", "g++"), "-std=c++17", "-g", "-fsanitize=address,undefined",
                    "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2407_04001_amd", "csrc"),
                    str(src), lib, "-Wl,-rpath," + os.path.dirname(lib), "-o", exe], check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120,
                       env=dict(os.environ, ASAN_OPTIONS="detect_leaks=0:abort_on_error=1"))
    assert r.returncode == 0 and expect in r.stdout, (r.returncode, (r.stdout + r.stderr)[-3000:])


def test_descriptors_stay_in_their_region(san_lib, tmp_path):
    """A launch descriptor outside the region that the memory layout made for
    its kind is refused before it is written, not put over the next region."""
    host_program(DESCRIPTORS, san_lib, tmp_path, "descriptors ok")


def test_caller_given_costs_keep_the_structure(san_lib, tmp_path):
    host_program(OVERRIDE, san_lib, tmp_path, "override ok")


def test_memory_limits_that_the_dense_fills_meet(san_lib, tmp_path):
    host_program(LIMITS, san_lib, tmp_path, "limits ok")
