"""Host-only checks of the C-ABI library: it loads, exports every symbol the header declares,
and rejects bad arguments before touching the GPU (so these run without one)."""
import ctypes as C
import os
import re

import numpy as np
import pytest

from paper_2408_08696_amd import synth, tr

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(tr.LIB_PATH):
        import __graft_entry__ as g
        g.build()
    return tr.lib()


def test_exports_match_header(lib):
    hdr = open(os.path.join(ROOT, "include", "tr.h")).read()
    declared = set(re.findall(r"\b(tr_[a-z_]+)\s*\(", hdr))
    assert declared == set(tr.EXPORTS)
    for name in declared:
        assert getattr(lib, name) is not None


def test_struct_layout_matches_header():
    assert C.sizeof(tr.StepOut) == 4 * (5 + 2 * tr.TR_MAX_LAYERS)
    assert C.sizeof(tr.Layer) == 9 * 8
    hdr = open(os.path.join(ROOT, "include", "tr.h")).read()
    assert f"#define TR_MAX_NODES {tr.TR_MAX_NODES}" in hdr
    assert f"#define TR_MAX_LAYERS {tr.TR_MAX_LAYERS}" in hdr
    assert f"#define TR_MAX_K {tr.TR_MAX_K}" in hdr


def test_strerror(lib):
    for s in (0, -1, -2, -3, -4, -5, -6, 7):
        assert lib.tr_strerror(s)


def _create(lib, V, k, parent, rank, n_layers):
    t, keep = tr.make_template(parent, rank, n_layers)
    h = C.c_void_p()
    return lib.tr_create(V, k, C.byref(t), C.byref(h)), h


@pytest.mark.parametrize("args,want", [
    ((0, 8, [-1], [-1], 1), tr.TR_EINVAL),
    ((10, 0, [-1], [-1], 1), tr.TR_EINVAL),
    ((10, 33, [-1], [-1], 1), tr.TR_EINVAL),
    ((10, 8, [0], [-1], 1), tr.TR_ETEMPLATE),                      # root parent must be -1
    ((10, 8, [-1, 1], [-1, 0], 2), tr.TR_ETEMPLATE),               # parent must precede child
    ((10, 8, [-1, 0], [-1, 8], 2), tr.TR_ETEMPLATE),               # rank >= k
    ((10, 8, [-1, 0, 0], [-1, 1, 1], 2), tr.TR_ETEMPLATE),         # duplicate (parent, rank)
    ((10, 8, [-1, 0, 1, 0], [-1, 0, 0, 1], 3), tr.TR_ETEMPLATE),   # not layer-major
    ((10, 8, [-1, 0], [-1, 0], 3), tr.TR_ETEMPLATE),               # n_layers disagrees
    ((10, 8, [-1] + list(range(128)), [-1] + [0] * 128, 129), tr.TR_ETEMPLATE),  # N > 128
])
def test_create_rejects_before_any_gpu_call(lib, args, want):
    st, h = _create(lib, *args)
    assert st == want and not h.value


def test_null_arguments(lib):
    assert lib.tr_create(10, 8, None, None) == tr.TR_EINVAL
    assert lib.tr_destroy(None) == tr.TR_EINVAL
    assert lib.tr_build_tree(None, None, None, None) == tr.TR_EINVAL
    assert lib.tr_matrix_load(None, None) == tr.TR_EINVAL
    assert lib.tr_verify_forward(None, None, None, None, None, None, None, 0, None) == tr.TR_EINVAL
    assert lib.tr_accept_and_update(None, None, None, None, None, None, None) == tr.TR_EINVAL
    assert lib.tr_prefill(None, None, None, None, 0, None, 0, None) == tr.TR_EINVAL
    assert lib.tr_op_topk(None, None, 0, 0, None, None) == tr.TR_EINVAL
    assert lib.tr_set_update_mode(None, 0) == tr.TR_EINVAL


def test_default_templates_are_accepted_by_the_host_check():
    # derive the same facts the library derives, from the header's rules, for all shipped templates
    for name, f in synth.TEMPLATES.items():
        t = f()
        assert t.parent[0] == -1 and t.rank[0] == -1
        assert all(0 <= t.parent[i] < i for i in range(1, t.n_nodes))
        assert t.n_nodes <= tr.TR_MAX_NODES and t.n_layers <= tr.TR_MAX_LAYERS


# ---- launch planners (host logic only) ----
def _variant_exists(nt, p, fused):
    """Kernel variants the projection source instantiates, by weight tiles per workgroup."""
    wt = 2 * p if fused else p
    if wt == 8:
        return nt in (4, 5)
    if wt == 6:
        return True
    if wt == 5:
        return not fused and nt <= 5
    return wt in ((2, 4) if fused else (1, 2, 3, 4))


@pytest.mark.parametrize("fused", [False, True])
def test_projection_plans_cover_every_tile_once(lib, fused):
    for n in (1, 15, 16, 17, 48, 64, 80, 81, 96, 112, 128):
        for in_f, out_f in ((256, 256), (4096, 4096), (4096, 12288), (4096, 11008), (11008, 4096), (5120, 13824),
                            (8192, 28672), (28672, 8192), (4096, 32000), (4096, 128256), (64, 32), (288, 96)):
            for ms in (1, 2, 4):
                p, groups, splits = tr.plan_projection(n, in_f, out_f, fused, ms)
                tiles = out_f // 16
                assert _variant_exists((n + 15) // 16, p, fused), (n, in_f, out_f, p)
                assert 1 <= groups <= tiles and groups * p >= tiles       # each tile has exactly one owner
                assert -(-tiles // groups) <= p                             # largest share fits the variant
                assert splits in (1, 2, 4) and splits <= (1 if fused else ms)
                assert splits == 1 or (in_f // 32) // splits >= 8           # every wave keeps >= 1 k-tile


def test_projection_plan_rejects_bad_shapes(lib):
    plan = (C.c_int32 * 3)()
    assert lib.tr_plan_projection(80, 4096, 4096, 0, 4, None) == tr.TR_EINVAL
    assert lib.tr_plan_projection(0, 4096, 4096, 0, 4, plan) == tr.TR_EINVAL
    assert lib.tr_plan_projection(129, 4096, 4096, 0, 4, plan) == tr.TR_EINVAL
    assert lib.tr_plan_projection(80, 4100, 4096, 0, 4, plan) == tr.TR_EINVAL
    assert lib.tr_plan_projection(80, 4096, 4100, 0, 4, plan) == tr.TR_EINVAL
    assert lib.tr_plan_projection(80, 4096, 4096, 0, 0, plan) == tr.TR_EINVAL


@pytest.mark.parametrize("n,in_f,out_f,splits,plan", [
    # op_linear stores its sums: that a step's o could save a launch by staying whole is no reason for it to take more workgroups.  One round
    (20, 4096, 4096, 2, (2, 128)), (1, 3200, 3200, 2, (2, 100)), (32, 3200, 3200, 4, (4, 50)), (20, 6656, 6656, 2, (4, 104)),
    (20, 4096, 4096, 1, (1, 256)), (80, 4096, 4096, 4, (4, 64))])
def test_linear_plans(lib, n, in_f, out_f, splits, plan):
    assert tr.plan_linear(n, in_f, out_f, splits) == plan and plan[1] * splits <= 256


def test_linear_plan_rejects_bad_shapes(lib):
    plan = (C.c_int32 * 2)()
    f = lib.tr_plan_linear
    assert f(80, 4096, 4096, 2, None) == tr.TR_EINVAL and f(0, 4096, 4096, 2, plan) == tr.TR_EINVAL
    assert f(129, 4096, 4096, 2, plan) == tr.TR_EINVAL and f(80, 4100, 4096, 2, plan) == tr.TR_EINVAL
    assert f(80, 4096, 4100, 2, plan) == tr.TR_EINVAL and f(80, 4096, 4096, 0, plan) == tr.TR_EINVAL
    assert f(80, 4096, 4096, 5, plan) == tr.TR_EINVAL


def test_projection_plans_of_the_7b_step_fill_the_chip(lib):
    # the five projections of a 7B layer at the 80-node tree: every plan puts work on >= 230 of 256 CUs
    for in_f, out_f, fused, ms in ((4096, 12288, False, 1), (4096, 4096, False, 4), (4096, 11008, True, 1),
                                   (11008, 4096, False, 4), (4096, 32000, False, 1)):
        p, groups, splits = tr.plan_projection(80, in_f, out_f, fused, ms)
        assert groups * splits >= 230, (in_f, out_f, p, groups, splits)


def test_step_projection_plan_rejects_bad_shapes(lib):
    plan = (C.c_int32 * 4)()
    f = lib.tr_plan_step_projection
    assert f(1, 80, 4096, 4096, None) == tr.TR_EINVAL
    assert f(-1, 80, 4096, 4096, plan) == tr.TR_EINVAL and f(4, 80, 4096, 4096, plan) == tr.TR_EINVAL
    assert f(1, 0, 4096, 4096, plan) == tr.TR_EINVAL and f(1, 129, 4096, 4096, plan) == tr.TR_EINVAL
    assert f(1, 80, 4100, 4096, plan) == tr.TR_EINVAL and f(1, 80, 4096, 4100, plan) == tr.TR_EINVAL


@pytest.mark.parametrize("projection", tr.PROJECTIONS)
def test_step_projection_plans_cover_every_tile_and_k_step_once(lib, projection):
    for n in (1, 16, 17, 33, 49, 65, 80, 81, 97, 128):
        for in_f in (64, 4096, 4160, 5120, 8192, 11008, 16384, 28672):
            for out_f in (32, 4096, 6432, 8192, 9632, 11008, 12832, 25632, 28672, 32000, 51232, 64000, 80000, 128256):
                tiles, pair = out_f // 16, projection == "gate_up"
                p, groups, splits, kernel = tr.plan_step_projection(projection, n, in_f, out_f)
                ms = 4 if projection == "o_down" else 1
                assert 1 <= splits <= ms and 1 <= groups <= tiles
                assert groups * p >= tiles and -(-tiles // groups) <= p       # one owner a tile, no share beyond the variant
                if kernel == 0:
                    assert (p, groups, splits) == tr.plan_projection(n, in_f, out_f, pair, ms)
                    continue
                assert projection != "qkv" and in_f >= 4096                   # the rest was not measured
                assert p * (2 if pair else 1) in ((6, 8, 16) if pair else (8, 16))
                per_k = -(-(in_f // 32) // splits)
                assert (splits - 1) * per_k < in_f // 32                      # no share of k is empty
                assert splits == 1 or per_k >= 128                            # shorter chains in the decode kernel, see below
                assert p * 2 != 6 or not pair or (in_f // 32) % 2 == 0        # its two groups of waves take the same k-steps
                wgs = groups * splits
                assert wgs >= -(-wgs // 256) * 200


@pytest.mark.parametrize("projection,in_f,out_f,out_tiles,shared,decode", [
    # rows for which a matrix shares operands in LDS, 16, 8 or 6 out-tiles a workgroup, and for which the decode kernel is as fast or
    # faster: one round of 16 out-tiles, few groups of them and many, ...
    ("gate_up", 8192, 28672, 16, (17, 32, 33, 64, 128), (1, 15, 16)), ("gate_up", 8192, 32768, 16, (33, 48, 80, 128), (1, 16, 17, 32)),
    ("gate_up", 4096, 28672, 16, (33, 49, 65, 128), (1, 16, 32)), ("lm_head", 4096, 64000, 16, (33, 64, 128), (1, 16, 17, 32)),
    ("lm_head", 5120, 51200, 16, (17, 32, 48, 128), (1, 16)), ("lm_head", 8192, 64000, 16, (33, 128), (1, 16, 32)),
    # ... several rounds, ...
    ("lm_head", 8192, 128256, 16, (33, 49, 80, 128), (1, 16, 32)), ("lm_head", 4096, 128256, 16, (49, 64, 80, 128), (1, 16, 32, 48)),
    # ... 8 out-tiles, ...
    ("lm_head", 4096, 32000, 8, (81, 96, 128), (1, 16, 33, 48, 49, 64, 80)), ("lm_head", 5120, 32000, 8, (33, 48, 81, 128), (1, 16, 32, 49, 64, 80)),
    ("gate_up", 5120, 13824, 8, (33, 48, 65, 80, 128), (1, 16, 17, 32, 49, 64)), ("gate_up", 8192, 16384, 8, (48, 81, 128), (1, 32, 64, 80)),
    ("gate_up", 4096, 14720, 8, (65, 80, 128), (1, 48, 64)), ("gate_up", 4096, 14784, 8, (81, 128), (48, 80)),
    ("lm_head", 8192, 80000, 8, (81, 128), (1, 16, 32, 48, 64, 80)),
    # ... 6, and matrices that do not fill the chip, or of short rows
    ("gate_up", 4096, 11008, 6, (97, 112, 128), (1, 80, 81, 96)), ("gate_up", 8192, 22016, 6, (97, 128), (64, 80, 96)),
    ("gate_up", 4128, 11008, 6, (), (97, 128)), ("lm_head", 4096, 25440, 8, (), (80, 128)), ("lm_head", 4064, 32000, 8, (), (80, 128)),
    ("qkv", 8192, 51200, 16, (), (1, 80, 128))])
def test_projections_that_share_operands(lib, projection, in_f, out_f, out_tiles, shared, decode):
    for n in shared:
        p, _, splits, kernel = tr.plan_step_projection(projection, n, in_f, out_f)
        assert (p * (2 if projection == "gate_up" else 1), splits, kernel) == (out_tiles, 1, 1), n
    for n in decode:
        assert tr.plan_step_projection(projection, n, in_f, out_f)[3] == 0, n


@pytest.mark.parametrize("in_f,heads,kv_heads,splits,split,whole", [
    # rows for which Q/K/V is taken in shares of k: as many as make 200 to 256 workgroups of 8 out-tiles, and for which it stays whole
    (8192, 64, 8, 3, (33, 48, 80, 128), (1, 16, 32)), (8192, 40, 8, 4, (33, 49, 65, 128), (1, 32)), (5120, 40, 40, 2, (97, 128), (1, 33, 80, 81, 96)),
    # (two shares from one row tile later on than three and four, and with fewer rows never)
    (7168, 56, 28, 2, (81, 128), (80,)), (8192, 64, 32, 2, (81, 128), (33, 64, 80)), (7168, 56, 8, 3, (81, 128), (80,)),
    (5120, 40, 8, 4, (81, 128), (1, 80)), (6144, 48, 8, 4, (81, 128), (33, 80)), (4096, 32, 32, 0, (), (1, 80, 128)),
    (5152, 40, 40, 2, (97, 128), (80, 81, 96)), (6144, 48, 48, 0, (), (80, 128)), (8192, 64, 64, 0, (), (33, 128))])
def test_qkv_in_shares_of_k(lib, in_f, heads, kv_heads, splits, split, whole):
    tiles = (heads + 2 * kv_heads) * 8
    for n in split:
        p, groups, s, kernel = tr.plan_step_qkv(n, in_f, heads, kv_heads)
        assert (p, groups, s, kernel) == (8, -(-tiles // 8), splits, 1) and 200 <= groups * s <= 256, n
        per_k = -(-(in_f // 32) // s)
        assert (s - 1) * per_k < in_f // 32                                       # no share of k is empty
        assert tr.plan_step_qkv(n, in_f, heads, kv_heads, tiled=False)[2:] == (1, 0), n
    for n in whole:
        assert tr.plan_step_qkv(n, in_f, heads, kv_heads) == tr.plan_step_projection("qkv", n, in_f, tiles * 16), n
        assert tr.plan_step_qkv(n, in_f, heads, kv_heads)[2:] == (1, 0), n
    assert tr.plan_step_qkv(128, in_f, heads, kv_heads, head_dim=64)[2:] == (1, 0)   # the kernel behind is for head dimension 128


def test_step_qkv_plan_rejects_bad_shapes(lib):
    plan = (C.c_int32 * 4)()
    f = lib.tr_plan_step_qkv
    assert f(80, 4096, 32, 32, 128, 1, None) == tr.TR_EINVAL and f(0, 4096, 32, 32, 128, 1, plan) == tr.TR_EINVAL
    assert f(129, 4096, 32, 32, 128, 1, plan) == tr.TR_EINVAL and f(80, 4100, 32, 32, 128, 1, plan) == tr.TR_EINVAL
    assert f(80, 4096, 32, 5, 128, 1, plan) == tr.TR_EINVAL and f(80, 4096, 32, 0, 128, 1, plan) == tr.TR_EINVAL
    assert f(80, 4096, 32, 32, 0, 1, plan) == tr.TR_EINVAL and f(80, 4096, 32, 32, 258, 1, plan) == tr.TR_EINVAL
    assert f(80, 4096, 32, 32, 128, 2, plan) == tr.TR_EINVAL


def test_ingestion_plans_cover_every_tile_and_k_step_once(lib):
    for n in (129, 144, 300, 512, 513, 700, 1024, 1025, 2047, 2048):
        for in_f in (64, 256, 4096, 5120, 8192, 28672):
            for out_f in (32, 1056, 4096, 5120, 6656, 8192):
                rows, p, groups, splits = tr.plan_ingestion(n, in_f, out_f)
                assert (rows, p) in ((8, 8), (8, 12), (16, 8), (16, 12), (16, 16))
                assert groups == -(-(out_f // 16) // p) and 1 <= splits <= 4
                assert splits * -(-n // 16) * 16 <= 2048                              # room for partial sums
                assert splits == 1 or (splits - 1) * -(-(in_f // 32) // splits) < in_f // 32
    plan = (C.c_int32 * 4)()
    f = lib.tr_plan_ingestion
    assert f(512, 4096, 4096, None) == tr.TR_EINVAL and f(128, 4096, 4096, plan) == tr.TR_EINVAL
    assert f(2049, 4096, 4096, plan) == tr.TR_EINVAL and f(512, 32, 4096, plan) == tr.TR_EINVAL
    assert f(512, 4100, 4096, plan) == tr.TR_EINVAL and f(512, 4096, 4100, plan) == tr.TR_EINVAL
    assert f(512, 4096, 0, plan) == tr.TR_EINVAL


@pytest.mark.parametrize("in_f,out_f,shared,decode", [
    # rows for which o and down share operands in LDS, in four shares of k, and for which they do not: never where a wave of the decode
    # kernel has shorter chains of sums (an eighth of a share, against 16 k-steps), nor where it is the faster one
    (4096, 6656, (), (1, 16, 80, 128)), (6656, 6656, (), (80, 96, 128)), (8192, 8192, (), (1, 48, 80, 128)),
    (11008, 8192, (), (80, 128)), (16256, 8192, (), (80, 128)), (16384, 8192, (81, 96, 128), (1, 16, 48, 64, 80)),
    (28672, 8192, (81, 128), (1, 16, 17, 48, 80)), (28672, 6208, (), (80, 128))])
def test_projections_in_shares_of_k(lib, in_f, out_f, shared, decode):
    for n in shared:
        assert tr.plan_step_projection("o_down", n, in_f, out_f)[2:] == (4, 1), n
    for n in decode:
        assert tr.plan_step_projection("o_down", n, in_f, out_f)[3] == 0, n


def test_whole_o_and_down_of_few_rows(lib):
    # kept whole so that they update the residual stream themselves: with one out-tile a workgroup, not with two for its sake ...
    for n in (17, 20, 32):
        for d, whole in ((4096, True), (3840, True), (3968, False), (3584, False), (3200, False)):
            assert (tr.plan_step_projection("o_down", n, d, d)[1:] == (d // 16, 1, 0)) == whole, (n, d)
        for d in (6432, 6656, 7168, 7552):
            assert tr.plan_step_projection("o_down", n, d, d)[2:] == (2, 0), (n, d)
        # ... and not where shares of many features are that much faster
    for n in (1, 15, 16):
        for in_f, d, whole in ((9568, 3584, True), (18944, 3584, False), (9888, 3712, True), (8864, 3328, True), (8640, 3200, False)):
            assert (tr.plan_step_projection("o_down", n, in_f, d)[1:] == (d // 16, 1, 0)) == whole, (n, in_f, d)
    for n in (17, 20, 32):
        assert tr.plan_step_projection("o_down", n, 8192, 8192) == (2, 256, 1, 0), n    # the faster plan in any case


def test_step_projections_of_the_7b_step_fill_the_chip(lib):
    # what 80- and 128-node steps of the 7B shape launch: with 128 nodes gate/up and the LM head share operands in LDS
    for projection, in_f, out_f, kernel in (("qkv", 4096, 12288, 0), ("o_down", 4096, 4096, 0), ("gate_up", 4096, 11008, 1),
                                            ("o_down", 11008, 4096, 0), ("lm_head", 4096, 32000, 1)):
        for n, want in ((80, 0), (128, kernel)):
            p, groups, splits, k = tr.plan_step_projection(projection, n, in_f, out_f)
            assert groups * splits >= 230 and k == want, (projection, n, p, groups, splits, k)


def test_attention_plan(lib):
    plan = (C.c_int32 * 2)()
    assert lib.tr_plan_attention(32, 32, 80, 600, None) == tr.TR_EINVAL
    assert lib.tr_plan_attention(0, 1, 80, 600, plan) == tr.TR_EINVAL
    assert lib.tr_plan_attention(32, 0, 80, 600, plan) == tr.TR_EINVAL
    assert lib.tr_plan_attention(32, 5, 80, 600, plan) == tr.TR_EINVAL      # not a multiple
    assert lib.tr_plan_attention(32, 32, 0, 600, plan) == tr.TR_EINVAL
    assert lib.tr_plan_attention(32, 32, 129, 600, plan) == tr.TR_EINVAL
    assert lib.tr_plan_attention(32, 32, 80, 0, plan) == tr.TR_EINVAL
    for H, Hkv in ((1, 1), (8, 8), (32, 32), (40, 40), (64, 8), (32, 8), (4, 2), (12, 4), (256, 256)):
        for n in (1, 16, 80, 128):
            prev = 1
            for L in (1, 31, 32, 33, 64, 100, 600, 2048, 8192, 65536):
                hpw, ns = tr.plan_attention(H, Hkv, n, L)
                if ns < 0:                                            # few-rows form: the whole group in a workgroup
                    assert hpw == H // Hkv and n * hpw <= 128 and (hpw > 2 or L > 832)
                    assert -ns <= 32 and -ns <= -(-L // 32) and (ns == -1 or -ns * Hkv <= 256)
                    continue
                if ns == 0:                                           # one-launch form: short sequences only
                    assert hpw == 1 and L <= 832 and H // Hkv <= 2 and prev <= 1
                    continue
                assert hpw in (1, 2) and (H // Hkv) % hpw == 0       # heads of one workgroup share a K/V head
                assert ((n + 15) // 16) * hpw <= (12 if hpw == 2 else 8)   # one wave per (head, node tile)
                groups = H // hpw
                assert 1 <= ns <= 16
                assert ns == 1 or 2 * ns <= -(-L // 32)               # at least two 32-key tiles per split
                assert ns == 1 or groups * ns <= 256                  # at most one workgroup per CU
                assert ns >= prev                                     # never fewer splits for a longer context
                prev = ns
    assert tr.plan_attention(32, 32, 80, 600) == (1, 0)
    assert tr.plan_attention(32, 32, 80, 1104) == (1, 8)
    assert tr.plan_attention(64, 8, 80, 600)[1] >= 1                      # eight query heads per K/V head: split form
    assert tr.plan_attention(40, 40, 80, 2128) == (1, 6)
    assert tr.plan_attention(64, 8, 80, 4176)[0] == 2
    assert tr.plan_attention(64, 8, 15, 16015) == (8, -32)                # all eight heads of a group, 32 key shares
    assert tr.plan_attention(32, 32, 1, 2049) == (1, -8)
    assert tr.plan_attention(16, 2, 1, 100) == (8, -1)                    # one share: no merge pass


@pytest.mark.parametrize("H,Hkv,n,short,long_", [
    # lengths (committed + nodes) whose shares are 32-key tiles one after another, and steps of 64 keys: sixteen tiles a share with
    # two heads a workgroup and up to 80 nodes, ...
    (32, 32, 80, (840, 1104, 3840), (3841, 16080)), (8, 8, 80, (3072, 7680), (7681,)), (40, 40, 80, (1152, 2128, 2880), (2881, 4176)),
    (256, 256, 66, (), (840, 1500)), (64, 8, 48, (1536, 3840), (3841, 4096)), (64, 8, 80, (3840,), (3841, 4176)),
    (64, 8, 96, (3840,), (3841,)), (32, 8, 80, (7680,), (7681,)), (64, 8, 64, (3840,), (3841,)),
    # ... 24 up to 112 nodes, 40 beyond
    (32, 32, 81, (5888,), (5889,)), (32, 32, 112, (5888,), (5889,)), (64, 8, 112, (2944,), (2945,)),
    (32, 32, 128, (905, 1536, 9984), (9985, 16128)), (64, 8, 113, (4992,), (4993,))])
def test_long_share_attention_rule(lib, H, Hkv, n, short, long_):
    for L in short:
        assert tr.plan_attention_form(H, Hkv, n, L) == "short_shares", L
    for L in long_:
        assert tr.plan_attention_form(H, Hkv, n, L) == "long_shares", L


def test_attention_forms(lib):
    form = C.c_int32()
    assert lib.tr_plan_attention_form(32, 32, 80, 600, None) == tr.TR_EINVAL
    assert lib.tr_plan_attention_form(32, 5, 80, 600, C.byref(form)) == tr.TR_EINVAL
    assert tr.plan_attention_form(32, 32, 80, 600) == "one_launch"
    assert tr.plan_attention_form(64, 8, 15, 16015) == "few_rows" and tr.plan_attention_form(256, 256, 1, 900) == "few_rows"


@pytest.mark.parametrize("H,Hkv,n,few,split", [
    # lengths (committed + nodes) measured faster as few rows, and as key splits
    (64, 8, 1, (100, 840, 16000), (20, 600)), (64, 8, 4, (128, 1200, 3000), (20, 300, 600, 1000)),
    (64, 8, 8, (2000, 3000), (1420,)), (64, 8, 15, (4000, 16015), (2000, 3072)), (64, 8, 16, (4000, 16016), (3090, 100)),
    (32, 8, 8, (128, 3100), (20, 300, 600, 1500)), (32, 8, 4, (100, 4000), (600, 1000)),
    (24, 8, 4, (100, 840, 3000), (20, 600)), (24, 8, 10, (200, 1500), (20, 600)), (56, 8, 4, (200, 840, 1500), (20, 600)),
    (32, 2, 2, (100, 3000), (20, 600, 1000)), (40, 8, 1, (400, 800), (20, 768)),
    (16, 8, 8, (3090, 16000), (840, 1500, 2500)), (32, 16, 16, (5200, 16000), (1000, 4100)),
    (32, 32, 1, (840, 2040), ()), (32, 32, 16, (1000, 16000), ()), (32, 32, 32, (3000, 16000), (840, 1000, 1500, 2040)),
    (8, 8, 32, (5200,), (840, 2040)), (16, 16, 64, (16000,), (1000, 8300)), (32, 32, 64, (8000,), (4100,)),
    (32, 32, 65, (), (840, 16000)), (64, 8, 17, (), (100, 16000)), (32, 32, 1, (), (100, 832)), (16, 8, 3, (), (100, 832))])
def test_few_rows_attention_rule(lib, H, Hkv, n, few, split):
    for L in few:
        assert tr.plan_attention(H, Hkv, n, L)[1] < 0, (H, Hkv, n, L)
    for L in split:
        assert tr.plan_attention(H, Hkv, n, L)[1] >= 0, (H, Hkv, n, L)


def test_static_topk_validates_before_touching_the_gpu(lib):
    """The entry point that allocates nothing: argument errors and its size limits are reported
    from the host, before any HIP call."""
    buf = np.zeros(64, np.int32)
    p = buf.ctypes.data
    f = lib.tr_op_topk_static
    assert f(None, tr.TR_F32, 4, 64, 8, p, None) == tr.TR_EINVAL
    assert f(p, tr.TR_F32, 4, 64, 8, None, None) == tr.TR_EINVAL
    assert f(p, 7, 4, 64, 8, p, None) == tr.TR_EINVAL
    assert f(p, tr.TR_F32, -1, 64, 8, p, None) == tr.TR_EINVAL
    assert f(p, tr.TR_F32, 4, 0, 8, p, None) == tr.TR_EINVAL
    assert f(p, tr.TR_F32, 4, 4, 8, p, None) == tr.TR_EINVAL                      # k > V
    assert f(p, tr.TR_F32, 4, 64, 9, p, None) == tr.TR_ECAPACITY                  # more candidates than it takes
    assert f(p, tr.TR_F32, tr.TR_MAX_NODES + 1, 64, 8, p, None) == tr.TR_ECAPACITY
    assert f(p, tr.TR_F32, 4, 131073, 8, p, None) == tr.TR_ECAPACITY              # beyond the static scratch
    assert f(p, tr.TR_F32, 4, 7, 7, p, None) == tr.TR_ECAPACITY                   # V below the kernels' minimum


def test_create_rejects_more_candidates_than_tokens(lib):
    st, _ = _create(lib, 4, 8, [-1], [-1], 1)
    assert st == tr.TR_EINVAL
