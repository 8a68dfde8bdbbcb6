"""The rules that pick a kernel's form from a call's sizes (csrc/tk_plan.hpp), compiled
for the host: every order gives each piece of work to one workgroup, keeps a KV
sequence on one XCD where it says so, and lies where the measurements put it."""
import ctypes
import itertools
import os
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2603_04427_amd", "csrc")

RANKED, OWNED, BY_SEQUENCE = 0, 1, 2

QUERIES = r"""
#include "tk_plan.hpp"
using namespace tk;
extern "C" {
void projection(long M, long N, long K, int* out) {
    const ProjShape s = project_shape(M, N, K);
    const ProjTileSize t = project_tile(s);
    out[0] = t.columns;
    out[1] = t.tokens;
    out[2] = s == ProjShape::k128x128whole;
    out[3] = (int)project_tiles(M, N, K);
}
void place(int order, int block, int pairs, int n, int* out) {
    const Place p = place_workgroup(order, block, pairs, n);
    out[0] = p.pair;
    out[1] = p.rank;
}
int walks(int B, int Hq, int Hkv, int Sq, int Sk, int r, int dv, int causal, int slots) {
    return walk_order({B, Hkv, Hq / Hkv, Sq, Sk, r, dv, causal != 0}, slots);
}
int form(int B, int Hq, int Hkv, int Sq, int Sk, int r, int dv, int causal) {
    const PrefillForm f = prefill_form({B, Hkv, Hq / Hkv, Sq, Sk, r, dv, causal != 0});
    return f.waves * 10 + f.groups;
}
int dq(int B, int Hq, int Hkv, int Sq, int Sk, int r, int dv, int causal) {
    const DqForm f = dq_form({B, Hkv, Hq / Hkv, Sq, Sk, r, dv, causal != 0});
    return f.waves * 10 + f.groups;
}
int dkdv_shape(int B, int Hq, int Hkv, int Sq, int Sk, int r, int dv, int causal) {
    const DkdvForm f = dkdv_form({B, Hkv, Hq / Hkv, Sq, Sk, r, dv, causal != 0});
    return f.waves * 1000 + f.groups * 100 + f.rows;
}
int dkdv(int B, int Hq, int Hkv, int Sq, int Sk, int r, int dv, int causal, int KW) {
    return dkdv_order({B, Hkv, Hq / Hkv, Sq, Sk, r, dv, causal != 0}, KW);
}
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    src, lib = d / "queries.cpp", d / "queries.so"
    src.write_text(QUERIES)
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", "-I" + CSRC, str(src), "-o", str(lib)],
                   check=True)
    return ctypes.CDLL(str(lib))


def places(plan, order, pairs, n):
    out = (ctypes.c_int * 2)()
    for block in range(pairs * n):
        plan.place(order, block, pairs, n, out)
        yield block, out[0], out[1]


@pytest.mark.parametrize("order", [RANKED, OWNED, BY_SEQUENCE])
def test_every_order_places_each_walk_once(plan, order):
    for pairs, n in itertools.product((1, 3, 7, 8, 12, 16, 20, 24, 56, 64, 104), (1, 2, 3, 5, 8, 13, 64)):
        if order == OWNED and pairs % 8:
            continue
        seen = [(pair, rank) for _, pair, rank in places(plan, order, pairs, n)]
        assert sorted(seen) == [(p, r) for p in range(pairs) for r in range(n)]


@pytest.mark.parametrize("order", [RANKED, OWNED, BY_SEQUENCE])
def test_longest_walks_start_first_on_each_xcd(plan, order):
    """Ranks rise over an XCD's workgroups: over all its pairs, or pair by pair."""
    for pairs, n in ((8, 5), (16, 4), (24, 7), (56, 3)):
        for xcd in range(8):
            mine = [(pair, rank) for block, pair, rank in places(plan, order, pairs, n) if block % 8 == xcd]
            assert mine == sorted(mine, key=(lambda w: w) if order == BY_SEQUENCE else (lambda w: w[1]))


@pytest.mark.parametrize("B,Hq,Hkv", [(2, 64, 8), (8, 28, 4), (8, 40, 5), (16, 6, 1), (4, 48, 8), (24, 32, 2)])
def test_head_groups_of_a_kv_sequence_share_an_xcd(plan, B, Hq, Hkv):
    """Several head groups read the same K and V: no order that such a call takes may spread
    them over the XCDs while the pairs divide among these."""
    G = Hq // Hkv
    per_kv = G // next(h for h in (4, 2, 1) if G % h == 0)
    pairs = B * Hkv * per_kv
    assert per_kv > 1 and pairs % 8 == 0
    for S, causal, r in itertools.product((300, 1000, 4096), (0, 1), (32, 128)):
        order = plan.walks(B, Hq, Hkv, S, S, r, 128, causal, 3 if r == 32 else 2)
        n = -(-S // 128)
        xcds = {}
        for block, pair, _ in places(plan, order, pairs, n):
            xcds.setdefault(pair // per_kv, set()).add(block % 8)
        # an eighth of the pairs may end inside a sequence: it then has two neighbours' XCDs
        assert sum(len(x) for x in xcds.values()) <= len(xcds) + 7


@pytest.mark.parametrize("call,slots,order", [
    ((2, 32, 8, 4096, 4096, 32, 128, 1), 3, RANKED),
    ((2, 32, 8, 8192, 8192, 32, 128, 1), 3, RANKED),
    ((4, 32, 8, 8192, 8192, 32, 128, 1), 3, BY_SEQUENCE),    # K and V over 6 MB an XCD, blocks fill it
    ((8, 32, 8, 6400, 6400, 32, 128, 1), 3, BY_SEQUENCE),
    ((4, 64, 8, 8192, 8192, 32, 128, 1), 3, BY_SEQUENCE),
    ((2, 64, 8, 4096, 4096, 32, 128, 1), 3, OWNED),
    ((4, 32, 32, 8192, 8192, 32, 128, 1), 3, BY_SEQUENCE),   # 42 MB an XCD, one head per KV sequence
    ((2, 32, 32, 8192, 8192, 32, 128, 1), 3, RANKED),        # 21 MB
    ((8, 32, 32, 2048, 2048, 32, 128, 0), 3, BY_SEQUENCE),   # equal walks
    ((4, 32, 32, 4096, 4096, 32, 128, 0), 3, BY_SEQUENCE),
    ((16, 32, 8, 1024, 1024, 32, 128, 0), 3, BY_SEQUENCE),
    ((1, 12, 12, 8192, 8192, 16, 64, 1), 3, RANKED),
    ((9, 28, 4, 5381, 5381, 32, 128, 1), 3, BY_SEQUENCE),    # 252 pairs, G 7, 7.8 MB
    ((2, 40, 5, 6000, 6000, 32, 128, 1), 3, RANKED),         # 20 pairs, 2.4 MB
    ((25, 40, 5, 123, 127, 128, 128, 1), 2, BY_SEQUENCE),
])
def test_order_of_measured_calls(plan, call, slots, order):
    assert plan.walks(*call, slots) == order


@pytest.mark.parametrize("call,order", [
    ((2, 32, 8, 4096, 4096, 32, 128, 1), RANKED),
    ((4, 32, 8, 8192, 8192, 32, 128, 1), BY_SEQUENCE),
    ((4, 32, 8, 8192, 8192, 128, 128, 1), RANKED),
    ((19, 32, 32, 2295, 2295, 32, 128, 0), BY_SEQUENCE),
])
def test_dkdv_order_of_measured_calls(plan, call, order):
    assert plan.dkdv(*call, 4) == order
    assert plan.dkdv(*call, 2) == RANKED  # two keys blocks a workgroup: few of them


@pytest.mark.parametrize("call,form", [
    ((1, 32, 8, 128, 8192, 32, 128, 1), 14),
    ((1, 32, 8, 500, 7700, 32, 128, 1), 24),
    ((1, 32, 8, 500, 7700, 128, 128, 1), 22),
    ((1, 32, 8, 1000, 8000, 32, 128, 1), 42),
    ((1, 32, 8, 1100, 1100, 32, 128, 1), 22),
    ((1, 32, 8, 2048, 2048, 32, 128, 1), 22),
    ((1, 12, 12, 4096, 4096, 32, 64, 1), 22),
    ((2, 32, 8, 1024, 1024, 32, 128, 1), 41),
    ((4, 32, 8, 512, 512, 32, 128, 1), 41),
    ((5, 32, 8, 207, 207, 32, 128, 1), 41),      # 4 tiles in 560 workgroups of two units
    ((5, 32, 8, 265, 265, 32, 128, 1), 41),
    ((15, 28, 4, 71, 71, 32, 128, 1), 41),       # G 7: rows past the end in every workgroup
    ((11, 6, 1, 244, 244, 32, 128, 1), 22),      # 4 tiles in 264 workgroups: one round
    ((5, 32, 32, 94, 94, 64, 128, 0), 41),       # 320 workgroups that fill a CU each
    ((7, 28, 4, 131, 508, 32, 128, 0), 41),      # equal walks in 392 workgroups of four units
    ((4, 8, 2, 1024, 1086, 32, 128, 0), 42),     # in 256
    ((4, 32, 4, 169, 169, 64, 64, 0), 41),       # equal walks of 3 tiles, all resident whole
    ((3, 32, 4, 225, 225, 16, 64, 1), 22),
    ((9, 32, 4, 158, 158, 64, 64, 1), 41),       # 720 workgroups of two units, two a CU
    ((15, 12, 12, 188, 1995, 64, 64, 1), 41),    # 540, equal walks
    ((5, 28, 4, 71, 108, 32, 128, 1), 41),       # 2 tiles in 280 workgroups
    ((4, 32, 8, 8192, 8192, 32, 128, 1), 41),
    ((1, 32, 8, 64, 64, 32, 128, 1), 41),        # one tile
])
def test_prefill_form_of_measured_calls(plan, call, form):
    assert plan.form(*call) == form


@pytest.mark.parametrize("call,form", [
    ((1, 32, 8, 512, 512, 32, 128, 1), 22),
    ((1, 32, 8, 1024, 1024, 128, 128, 1), 22),
    ((2, 12, 12, 2048, 2048, 32, 64, 1), 22),
    ((1, 32, 8, 2048, 2048, 32, 128, 1), 42),
    ((3, 32, 32, 500, 500, 32, 128, 1), 41),
    ((2, 32, 8, 4096, 4096, 32, 128, 1), 41),
    ((5, 28, 4, 104, 104, 64, 128, 1), 41),      # short walks in more workgroups than one a CU
    ((4, 28, 4, 134, 134, 64, 128, 1), 41),
    ((11, 32, 8, 47, 65, 32, 128, 1), 41),
    ((7, 32, 8, 125, 125, 32, 128, 1), 41),
    ((2, 32, 8, 374, 374, 32, 128, 1), 22),
    ((10, 32, 8, 86, 447, 64, 128, 1), 41),      # equal walks
    ((15, 12, 12, 184, 184, 64, 64, 0), 41),
    ((6, 8, 2, 375, 761, 128, 128, 0), 42),      # equal and long, four units in 144 workgroups
    ((2, 8, 2, 2684, 2684, 32, 128, 0), 41),
    ((1, 12, 12, 5129, 5129, 32, 64, 0), 42),
    ((1, 32, 8, 33, 33, 32, 128, 1), 41),        # one tile
])
def test_dq_form_of_measured_calls(plan, call, form):
    assert plan.dq(*call) == form


@pytest.mark.parametrize("call,form", [
    ((1, 32, 8, 1024, 1024, 32, 128, 1), 2432),
    ((1, 32, 8, 2048, 2048, 32, 128, 1), 2432),
    ((2, 32, 8, 4096, 4096, 32, 128, 1), 2232),
    ((9, 8, 2, 1513, 1713, 32, 128, 1), 2432),
    ((4, 32, 8, 600, 600, 32, 128, 1), 2432),
    ((9, 32, 8, 277, 277, 32, 128, 1), 2432),
    ((13, 32, 8, 411, 411, 32, 128, 0), 2232),
    ((1, 12, 12, 4096, 4096, 32, 64, 1), 2264),
    ((2, 32, 4, 2395, 2395, 32, 64, 1), 2432),
    ((15, 16, 16, 99, 166, 32, 64, 1), 4164),
    ((10, 32, 4, 1132, 1132, 32, 64, 0), 2264),
    ((1, 12, 12, 1716, 1716, 64, 64, 1), 2432),
    ((6, 32, 8, 645, 645, 128, 128, 1), 2264),
    ((1, 32, 32, 659, 669, 64, 128, 1), 2264),
    ((1, 32, 32, 512, 518, 64, 128, 1), 2264),
    ((1, 32, 4, 591, 591, 32, 64, 1), 2432),
    ((1, 32, 8, 2048, 2048, 128, 128, 1), 2264),
    ((4, 32, 8, 4096, 4096, 32, 128, 1), 4164),
    ((1, 32, 32, 2048, 2048, 128, 128, 1), 4164),
    ((8, 12, 12, 1000, 1000, 32, 64, 1), 4164),
    ((4, 32, 32, 153, 169, 32, 128, 0), 2232),   # 384 workgroups of two units: not x 4
    ((13, 32, 32, 104, 104, 32, 128, 0), 4164),  # equal walks, a second round
    ((7, 64, 8, 877, 877, 32, 128, 0), 4164),
    ((13, 32, 8, 157, 157, 128, 128, 0), 4164),
    ((11, 40, 5, 43, 492, 128, 128, 1), 4164),
    ((9, 16, 16, 267, 267, 32, 64, 0), 4164),
    ((1, 32, 32, 40, 4096, 32, 128, 1), 4164),   # one query tile a walk
])
def test_dkdv_form_of_measured_calls(plan, call, form):
    assert plan.dkdv_shape(*call) == form


# calls of all sizes, to see which forms a width can take
CALLS = [(B, Hkv * G, Hkv, Sq, Sk, causal) for B in (1, 3, 16) for Hkv in (1, 8, 32) for G in (1, 4, 7)
         for Sq, Sk in ((1, 1), (60, 60), (60, 3000), (130, 190), (300, 300), (700, 1400), (1100, 1100), (2500, 2500),
                        (8192, 8192)) for causal in (0, 1)]


def test_prefill_shapes_of_the_parity_tests_cover_every_form_and_order(plan):
    from test_gpu_prefill import ORDERS, WORKGROUP_SHAPES, WORKGROUP_WIDTHS
    names = {"longest first": RANKED, "owned": OWNED, "by sequence": BY_SEQUENCE}
    for r, dv in WORKGROUP_WIDTHS:
        tested = {plan.form(*call[:5], r, dv, call[5]) for call in WORKGROUP_SHAPES}
        assert tested | {41} == {plan.form(*call[:5], r, dv, call[5]) for call in CALLS}, (r, dv)
    for r, dv in [(32, 64), *WORKGROUP_WIDTHS]:
        for call, order in ORDERS:
            assert plan.form(*call[:5], r, dv, call[5]) == 41, (call, r, dv)
            assert plan.walks(*call[:5], r, dv, call[5], 3 if r <= 32 else 2) == names[order], (call, r, dv)
    assert {order for _, order in ORDERS} == set(names)


def test_backward_shapes_of_the_parity_tests_cover_every_form_and_order(plan):
    from test_gpu_backward import ORDERS, WORKGROUP_SHAPES, WORKGROUP_WIDTHS
    names = {"longest first": RANKED, "owned": OWNED, "by sequence": BY_SEQUENCE}
    for width in WORKGROUP_WIDTHS:
        for query in (plan.dq, plan.dkdv_shape):
            tested = {query(*call[:5], r, dv, call[5]) for r, dv, call in WORKGROUP_SHAPES if (r, dv) == width}
            assert tested == {query(*call[:5], *width, call[5]) for call in CALLS}, (width, query.__name__)
        for call, order in ORDERS:
            assert plan.dq(*call[:5], *width, call[5]) == 41, (call, width)
            assert plan.walks(*call[:5], *width, call[5], 2) == names[order], (call, width)
        whole = {call for call, _ in ORDERS if plan.dkdv_shape(*call[:5], *width, call[5]) == 4164}
        assert {plan.dkdv(*call[:5], *width, call[5], 4) for call in whole} == {RANKED, BY_SEQUENCE}, width


def test_projection_shapes_of_the_parity_test_cover_every_tile(plan):
    """Each entry of the GPU parity test runs the tile it is listed with, and every tile
    of the ladder has one."""
    from test_gpu_project import SHAPES
    out = (ctypes.c_int * 4)()
    for (B, S, d_model, heads, width), tile in SHAPES:
        plan.projection(ctypes.c_long(B * S), ctypes.c_long(heads * width), ctypes.c_long(d_model), out)
        assert f"{out[0]}x{out[1]}" + (" whole" if out[2] else "") == tile, (B, S, d_model, heads, width)
        assert out[3] == -(-B * S // out[1]) * -(-heads * width // out[0])
    assert {tile for _, tile in SHAPES} == {"16x16", "16x32", "32x32", "32x64", "64x64", "64x128", "128x64", "128x128",
                                            "128x128 whole", "256x128", "256x256"}


@pytest.mark.parametrize("M,N,K,tile", [
    (16, 1024, 4096, "16x16"),
    (200, 2048, 4096, "64x64"),
    (418, 768, 4096, "64x64"),        # 168 tiles of 32 x 64
    (2035, 256, 768, "32x64"),        # 256 of them
    (255, 2048, 1536, "64x64"),
    (1500, 1024, 4096, "64x128"),
    (2202, 768, 768, "128x64"),
    (1400, 3072, 4096, "128x128 whole"),
    (3004, 2048, 4096, "128x128 whole"),
    (6276, 1024, 4096, "256x128"),    # 8 MiB of weights
    (12534, 512, 4096, "256x128"),
    (3000, 4096, 4096, "256x256"),
    (4500, 4096, 4096, "256x128"),    # 288 tiles of 256 x 256
    (32768, 1024, 4096, "256x256"),
])
def test_projection_tile_of_measured_calls(plan, M, N, K, tile):
    out = (ctypes.c_int * 4)()
    plan.projection(ctypes.c_long(M), ctypes.c_long(N), ctypes.c_long(K), out)
    assert f"{out[0]}x{out[1]}" + (" whole" if out[2] else "") == tile
