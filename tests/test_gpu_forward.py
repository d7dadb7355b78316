"""GPU parity of the verification forward and of whole decode steps against the oracle."""
import numpy as np
import pytest
import torch

from oracle import tr_oracle as O
from paper_2408_08696_amd import synth, tr
from gpu_util import kv_fill, kv_plain_views, lockstep, oracle_cfg, require_gpu, say, to_gpu
from test_oracle_loop import FIXTURE_MIN_GAP, fixture_min_gap

pytestmark = pytest.mark.gpu
K = 8


@pytest.mark.parametrize("tmpl_name", ["tree15", "tree15_alt", "single"])
def test_tiny_fp32_free_running(tmpl_name):
    """The small fp32 config end to end, free running: 64 new tokens; emitted tokens, trees,
    accepted lengths and M bit-exact, logits within 1e-4 absolute — and within a quarter of the
    smallest top-k gap of the run, so no decision could have flipped."""
    require_gpu()
    sh = synth.SHAPES["tiny"]
    tmpl = synth.TEMPLATES[tmpl_name]()
    w = synth.make_weights(sh, seed=0)
    wn = synth.weights_to_numpy(w)
    prompt = synth.zipf_prompt(sh.vocab, 64, seed=0, ngram=4).tolist()
    M0 = synth.init_matrix(sh.vocab, K)
    eng = tr.Engine(sh, to_gpu(w), tmpl, k=K, capacity=64 + 64 + tmpl.n_nodes + 8)
    eng.ctx.matrix_load(M0)
    eng.prefill(prompt)

    cfg = oracle_cfg(sh)
    tree = O.make_tree(tmpl.parent, tmpl.rank, K)
    M = M0.astype(np.int64)
    steps = []
    toks, lens, kv = O.tr_generate(cfg, wn, M, tree, prompt, 64, K, on_step=steps.append)
    M_run = M0.astype(np.int64)
    got, max_err = [], 0.0
    for i, r in enumerate(steps):
        say("tiny fp32", tmpl_name, "step", i)
        h = eng.step(sync=True)
        assert eng.S.cpu().tolist() == r.S.tolist(), f"step {i}: tree"
        max_err = max(max_err, float(np.abs(eng.logits.cpu().numpy() - r.logits).max()))
        assert np.array_equal(eng.topk.cpu().numpy(), r.topk), f"step {i}: top-k"
        assert h.n_accepted == r.acc.n_accepted and list(h.path[:h.n_emitted]) == r.acc.path
        assert list(h.emitted[:h.n_emitted]) == r.acc.emitted
        got.extend(h.emitted[:h.n_emitted])
        O.update_matrix(M_run, r.S, r.topk)
        assert np.array_equal(eng.ctx.matrix_store().astype(np.int64), M_run), f"step {i}: matrix"
    assert got[:64] == toks
    ar, _, _ = O.ar_generate(cfg, wn, prompt, 64)
    assert got[:64] == ar                                     # lossless on the GPU too
    say("max |logit error|", max_err)
    assert max_err < 1e-4
    if tmpl_name == "tree15":
        assert 4 * max_err < FIXTURE_MIN_GAP <= fixture_min_gap(0)
    # committed KV equals the oracle's cache (K as stored, V transposed)
    L = kv.len
    kp, vp = kv_plain_views(eng.kv)
    kg = kp[:, :, :L, :].permute(0, 2, 1, 3).cpu().numpy()
    vg = vp[:, :, :L, :].permute(0, 2, 1, 3).cpu().numpy()
    for l in range(sh.n_layers):
        assert np.abs(kg[l] - kv.k[l][:L]).max() < 1e-4 and np.abs(vg[l] - kv.v[l][:L]).max() < 1e-4


@pytest.mark.parametrize("shape_name,tmpl_name", [("tiny_bf16", "tree80"), ("tiny_gqa_bf16", "tree80"),
                                                  ("tiny_bf16", "tree81"), ("tiny_bf16", "wide128"),
                                                  ("tiny_bf16", "single"), ("tiny", "tree80"),
                                                  ("tiny_odd_bf16", "tree80"), ("tiny_bf16:rowmajor", "tree15"),
                                                  ("tiny_bf16", "prefix48"), ("tiny_gqa_bf16", "prefix97"),
                                                  # the depth sweep's 80-node templates of 4, 5, 7 and 8 layers
                                                  ("tiny_bf16", "depth4"), ("tiny_bf16", "depth5"),
                                                  ("tiny_gqa_bf16", "depth7"), ("tiny_bf16", "depth8"),
                                                  ("tiny_hd64_bf16", "tree80"), ("tiny_gqa_bf16:plainkv", "tree80"),
                                                  # projection-kernel variants of the full-size models
                                                  ("zoo_ffn5504", "tree80"), ("zoo_ffn5504", "tree81"),
                                                  ("zoo_ffn11008", "tree80"), ("zoo_ffn11008", "wide128"),
                                                  ("zoo_ffn11008", "single"), ("zoo_ffn13824", "tree80"),
                                                  ("zoo_ffn13824", "prefix64"), ("zoo_heads32", "tree80"),
                                                  ("zoo_heads40", "tree80"), ("zoo_heads32", "wide128")])
def test_small_shapes_lockstep(shape_name, tmpl_name):
    require_gpu()
    pack, kv_tiled = None, None
    if shape_name.endswith(":rowmajor"):
        shape_name, pack = shape_name.split(":")[0], False    # bf16 through the generic kernels
    if shape_name.endswith(":plainkv"):
        shape_name, kv_tiled = shape_name.split(":")[0], False  # packed projections, position-major cache
    sh = synth.SHAPES[shape_name]
    tmpl = (synth.prefix_template(int(tmpl_name[6:])) if tmpl_name.startswith("prefix")
            else synth.TEMPLATES[tmpl_name]())
    w = synth.make_weights(sh, seed=1)
    prompt = synth.zipf_prompt(sh.vocab, 150, seed=3, ngram=8).tolist()
    eng = tr.Engine(sh, to_gpu(w), tmpl, k=K, capacity=512, pack=pack, kv_tiled=kv_tiled)
    assert eng.model.packed == (tr.can_pack(sh) if pack is None else pack)
    assert eng.kv.tiled == ((sh.dtype == "bf16" and sh.head_dim == 128) if kv_tiled is None else kv_tiled)
    abs_tol = 1e-4 if sh.dtype == "f32" else None
    stats, _ = lockstep(eng, sh, synth.weights_to_numpy(w), tmpl, prompt, 6, synth.init_matrix(sh.vocab, K),
                        abs_tol=abs_tol, label=f"{shape_name}/{tmpl_name}")
    say(stats)


HOT_PLAN = [5, 1, 0, 5, 2, 0, 1, 3]


@pytest.mark.parametrize("shape_name,tmpl_name", [("tiny_bf16", "tree80"), ("tiny_gqa_bf16", "tree80"),
                                                  ("zoo_heads32", "tree80"), ("tiny_gqa_bf16:plainkv", "tree80"),
                                                  ("tiny_bf16", "wide128"), ("tiny", "tree15")])
def test_hot_started_lockstep_accepts_drafts(shape_name, tmpl_name):
    """Whole steps on the packed / matrix-core / tiled-cache path with drafts really accepted
    (Section 2.2 chain rule, Section 3.3): the matrix starts with the oracle's continuation of the
    prompt planted (Section 3.1 hot start), so steps accept 0, 1, ... depth-1 drafts, the accepted
    rows are compacted, and the next step attends over the compacted rows.  Every step is compared
    with the oracle, and so are the cache rows each step commits."""
    require_gpu()
    kv_tiled = None
    if shape_name.endswith(":plainkv"):
        shape_name, kv_tiled = shape_name.split(":")[0], False
    sh = synth.SHAPES[shape_name]
    tmpl = synth.TEMPLATES[tmpl_name]()
    plan = [tmpl.n_layers - 1 if a == 5 else min(a, tmpl.n_layers - 1) for a in HOT_PLAN]
    w = synth.make_weights(sh, seed=1)
    prompt = synth.zipf_prompt(sh.vocab, 150, seed=3, ngram=8).tolist()
    eng = tr.Engine(sh, to_gpu(w), tmpl, k=K, capacity=512, kv_tiled=kv_tiled)
    stats, _ = lockstep(eng, sh, synth.weights_to_numpy(w), tmpl, prompt, len(plan), synth.init_matrix(sh.vocab, K),
                        abs_tol=1e-4 if sh.dtype == "f32" else None, label=f"hot {shape_name}/{tmpl_name}",
                        hot_plan=plan, check_cache=True)
    say(stats)
    seen = {s["n_emitted"] - 1 for s in stats}
    assert {0, 1, tmpl.n_layers - 1} <= seen, seen


def test_hot_started_sampling_lockstep():
    """The same under temperature sampling (Section 5.3): the planted continuation is the oracle's
    sampled one (same per-position noise), so sampled drafts are accepted and compacted."""
    require_gpu()
    sh = synth.SHAPES["tiny_gqa_bf16"]
    tmpl = synth.tree80()
    w = synth.make_weights(sh, seed=4)
    prompt = synth.zipf_prompt(sh.vocab, 70, seed=4).tolist()
    noise = synth.gumbel_noise(70 + (len(HOT_PLAN) + 1) * tmpl.n_layers, sh.vocab, seed=9).numpy()
    eng = tr.Engine(sh, to_gpu(w), tmpl, k=K, capacity=70 + len(HOT_PLAN) * tmpl.n_layers + tmpl.n_nodes + 32)
    stats, _ = lockstep(eng, sh, synth.weights_to_numpy(w), tmpl, prompt, len(HOT_PLAN),
                        synth.init_matrix(sh.vocab, K), label="hot sampling", sampler=(1.0, noise),
                        hot_plan=HOT_PLAN, check_cache=True)
    say(stats)
    seen = {s["n_emitted"] - 1 for s in stats}
    assert {0, 1, tmpl.n_layers - 1} <= seen, seen


@pytest.mark.parametrize("shape_name,temperature", [("tiny", 0.8), ("tiny_bf16", 0.5), ("tiny_gqa_bf16", 1.0)])
def test_temperature_sampling_lockstep(shape_name, temperature):
    """Whole steps under temperature sampling (Section 5.3): drawn tokens, accept lengths, emitted
    tokens, the matrix and the cache length must follow the oracle's rule applied to the GPU's logits."""
    require_gpu()
    sh = synth.SHAPES[shape_name]
    tmpl = synth.tree80()
    w = synth.make_weights(sh, seed=4)
    wn = synth.weights_to_numpy(w)
    prompt = synth.zipf_prompt(sh.vocab, 70, seed=4).tolist()
    n_steps = 6
    eng = tr.Engine(sh, to_gpu(w), tmpl, k=K, capacity=70 + n_steps * tmpl.n_layers + tmpl.n_nodes + 32)
    noise = synth.gumbel_noise(70 + (n_steps + 1) * tmpl.n_layers, sh.vocab, seed=9).numpy()
    stats, _ = lockstep(eng, sh, wn, tmpl, prompt, n_steps, synth.init_matrix(sh.vocab, K),
                        abs_tol=1e-4 if sh.dtype == "f32" else None, label=f"{shape_name} T={temperature}",
                        sampler=(1.0 / temperature, noise))
    say(stats)


def test_prefill_crosses_chunk_boundaries():
    """A 300-token prompt goes through three chain chunks (128 + 128 + 43); the cache must equal
    the oracle's causal prefill."""
    require_gpu()
    sh = synth.SHAPES["tiny"]
    w = synth.make_weights(sh, seed=2)
    wn = synth.weights_to_numpy(w)
    prompt = synth.zipf_prompt(sh.vocab, 300, seed=1).tolist()
    eng = tr.Engine(sh, to_gpu(w), synth.tree15(), k=K, capacity=400)
    eng.prefill(prompt)
    torch.cuda.synchronize()
    assert int(eng.kv.d_len.item()) == 299 and eng.kv.c.len_bound == 299
    cfg = oracle_cfg(sh)
    kv = O.KVCache(cfg, 400)
    O.prefill(cfg, wn, kv, prompt[:-1])
    kp, vp = kv_plain_views(eng.kv)
    kg = kp[:, :, :299, :].permute(0, 2, 1, 3).cpu().numpy()
    vg = vp[:, :, :299, :].permute(0, 2, 1, 3).cpu().numpy()
    for l in range(sh.n_layers):
        assert np.abs(kg[l] - kv.k[l][:299]).max() < 1e-4
        assert np.abs(vg[l] - kv.v[l][:299]).max() < 1e-4


HEADS32 = synth.ModelShape("heads32", 2, 256, 32, 32, 128, 672, 2048, "bf16")
HEADS64_8 = synth.ModelShape("heads64_8", 2, 256, 64, 8, 128, 672, 2048, "bf16")


def _shape(name):
    return {"heads32": HEADS32, "heads64_8": HEADS64_8}.get(name) or synth.SHAPES[name]


def _smallest_workspace(eng):
    """Cuts the engine's workspace to what passes of 512 rows need."""
    sh = eng.shape  # bytes per row of the activation buffers: x, xn, q, attn, h, rope, ssq
    per_row = sh.d_model * 6 + sh.n_heads * sh.head_dim * 4 + sh.d_ffn * 2 + sh.head_dim * 4 + (sh.d_model + 1023) // 1024 * 4
    eng.ws = eng.ws[:eng.ws.numel() - 1536 * per_row]


def _cache_against_oracle(eng, kv, n):
    kp, vp = kv_plain_views(eng.kv, k_interleaved=True)
    kg = kp[:, :, :n, :].permute(0, 2, 1, 3).float().cpu().numpy()
    vg = vp[:, :, :n, :].permute(0, 2, 1, 3).float().cpu().numpy()
    for l in range(eng.shape.n_layers):
        # per row, so that a wrong row in one block cannot hide behind the largest entry of the whole cache
        dk = np.abs(kg[l] - kv.k[l][:n]).max(axis=(1, 2)) / np.abs(kv.k[l][:n]).max(axis=(1, 2))
        dv = np.abs(vg[l] - kv.v[l][:n]).max(axis=(1, 2)) / np.abs(kv.v[l][:n]).max(axis=(1, 2))
        say("layer", l, "relative K error", dk.max(), "at row", int(dk.argmax()), "V error", dv.max(), "at row",
            int(dv.argmax()))
        assert dk.max() < 2e-2 and dv.max() < 2e-2


@pytest.mark.parametrize("shape_name,plen,small", [("tiny_bf16", 100, False), ("tiny_bf16", 150, False),
                                                   ("tiny_gqa_bf16", 150, False), ("tiny_bf16", 513, False),
                                                   ("tiny_gqa_bf16", 600, False), ("tiny_bf16", 700, False),
                                                   ("zoo_heads32", 300, False), ("tiny_gqa_bf16", 1100, False),
                                                   ("tiny_bf16", 2049, False),
                                                   # several passes
                                                   ("tiny_gqa_bf16", 2101, False), ("tiny_gqa_bf16", 600, True),
                                                   ("tiny_bf16", 1100, True), ("tiny_bf16", 514, True)])
def test_packed_prefill_cache_matches_oracle(shape_name, plen, small):
    """Packed bf16 models rotate and store queries, keys and values in the epilogue of the fused Q/K/V
    projection; the committed cache must hold the oracle's keys (read back through the interleaved feature
    order of such models) and values, to bf16 accuracy.  With a tiled cache, prompts beyond 128 tokens go
    through the ingestion kernels in passes of up to 2048 rows, or 512 with the smallest workspace (`small`): the
    lengths cover one decode-path pass (99 rows), a ragged second row block (149), whole row blocks (512, 2048), ragged
    ones (599, 699, 1099), a single-layer model (only the Q/K/V projection runs), two wide passes (2100 = 1280 + 820),
    wide passes with a short one behind them that the decode kernels take (599 = 512 + 87, 513 = 512 + 1) and three
    (1099 = 512 + 512 + 75)."""
    require_gpu()
    say("packed prefill cache", shape_name, plen, small)
    sh = _shape(shape_name)
    w = synth.make_weights(sh, seed=2)
    wn = synth.weights_to_numpy(w)
    prompt = synth.zipf_prompt(sh.vocab, plen, seed=2).tolist()
    eng = tr.Engine(sh, to_gpu(w), synth.tree15(), k=K, capacity=plen + 106)
    assert eng.model.packed and eng.kv.tiled
    if small:
        _smallest_workspace(eng)
    eng.prefill(prompt)
    torch.cuda.synchronize()
    n = plen - 1
    assert int(eng.kv.d_len.item()) == n and eng.kv.c.len_bound == n
    kv = O.KVCache(oracle_cfg(sh), plen + 106)
    O.prefill(oracle_cfg(sh), wn, kv, prompt[:-1])
    _cache_against_oracle(eng, kv, n)


@pytest.mark.parametrize("d,heads,F,plen,tiles", [
    (1056, 2, 480, 150, (8, 8)), (4128, 2, 480, 300, (8, 8)), (6560, 2, 480, 522, (8, 12)), (4096, 2, 256, 2049, (16, 8)),
    (6144, 2, 256, 2049, (16, 12)), (8160, 2, 256, 2001, (16, 16)), (1056, 8, 2048, 497, None), (1056, 8, 2048, 498, None),
    (1056, 8, 2048, 540, None)])
def test_ingestion_that_updates_the_residual_stream(d, heads, F, plen, tiles):
    """o and down that are not split over k add to the residual stream in their own epilogue, in every workgroup shape, with out-tiles
    missing in the last workgroup and rows in the last block; with 8 heads they are split, and the residual kernel takes its rows one by
    one up to 31 row tiles and by eights from 32 on.  The second layer's keys and values carry what they leave, the operand and
    the sums of squares.  Gains are powers of two, so that they round nothing."""
    require_gpu()
    say("ingestion with residual epilogue", d, heads, F, plen)
    plans = [tr.plan_ingestion(plen - 1, in_f, d) for in_f in (heads * 128, F)]             # o and down
    if tiles is not None:
        assert all(p[:2] == tiles and p[3] == 1 for p in plans), plans
    else:
        assert all(p[3] > 1 for p in plans), plans
    sh = synth.ModelShape("resid", 2, d, heads, 1, 128, F, 512, "bf16")
    w = synth.make_weights(sh, seed=8)
    gen = torch.Generator().manual_seed(d)
    for lw in w["layers"]:
        for name in ("attn_norm", "ffn_norm"):
            lw[name] = (lw[name] * 2.0 ** torch.randint(-1, 2, (d,), generator=gen)).to(torch.bfloat16)
    prompt = synth.zipf_prompt(sh.vocab, plen, seed=8).tolist()
    eng = tr.Engine(sh, to_gpu(w), synth.tree15(), k=K, capacity=plen + 40)
    eng.prefill(prompt)
    torch.cuda.synchronize()
    kv = O.KVCache(oracle_cfg(sh), plen + 40, np.float32)
    O.prefill(oracle_cfg(sh), synth.weights_to_numpy(w), kv, prompt[:-1], np.float32)
    _cache_against_oracle(eng, kv, plen - 1)


@pytest.mark.parametrize("shape_name,lens", [("heads64_8", (131, 530)), ("heads32", (129, 1160))])
def test_ingestion_attention_forms_match_oracle(shape_name, lens):
    """The ingestion attention where a launch has more than one workgroup per compute unit (64 heads x 5 row blocks, 32 x
    10), two heads of a group in a workgroup or one head alone, behind an odd committed length: the second layer's keys
    and values carry its result, per row."""
    require_gpu()
    say("ingestion attention", shape_name, lens)
    sh = _shape(shape_name)
    w = synth.make_weights(sh, seed=7)
    wn = synth.weights_to_numpy(w)
    n = sum(lens)
    prompt = synth.zipf_prompt(sh.vocab, n + 1, seed=7).tolist()
    eng = tr.Engine(sh, to_gpu(w), synth.tree15(), k=K, capacity=n + 40)
    eng.prefill(prompt[:lens[0] + 1])
    eng.prefill(prompt[lens[0]:], keep_cache=True)
    torch.cuda.synchronize()
    assert int(eng.kv.d_len.item()) == n
    kv = O.KVCache(oracle_cfg(sh), n + 40, np.float32)
    O.prefill(oracle_cfg(sh), wn, kv, prompt[:n], np.float32)
    _cache_against_oracle(eng, kv, n)


@pytest.mark.parametrize("shape_name,lens", [("tiny_bf16", (2400,)), ("tiny_gqa_bf16", (2400,)), ("tiny_gqa_bf16", (131, 1000, 300)),
                                             ("heads32", (1100, 1030)), ("heads64_8", (650, 2101))])
def test_prefill_same_cache_with_the_smallest_workspace(shape_name, lens):
    """A workspace that holds 512 rows (what tr_workspace_bytes asked for before passes of 2048) is accepted and gives the
    cache that the full one gives: passes, K-splits and attention shapes (keys split over two waves, two heads of a
    group, one head) differ, the sums only in their order.  Runs of several calls start at odd committed lengths."""
    require_gpu()
    say("prefill workspace", shape_name, lens)
    sh = _shape(shape_name)
    w = to_gpu(synth.make_weights(sh, seed=6))
    prompt = synth.zipf_prompt(sh.vocab, sum(lens) + 1, seed=6).tolist()
    caches = []
    for small in (False, True):
        eng = tr.Engine(sh, w, synth.tree15(), k=K, capacity=sum(lens) + 40)
        if small:
            _smallest_workspace(eng)
        lo = 0
        for i, n in enumerate(lens):
            eng.prefill(prompt[lo:lo + n + 1], keep_cache=i > 0)
            lo += n
        assert int(eng.kv.d_len.item()) == lo
        caches.append((eng.kv.k.clone(), eng.kv.v.clone(), *kv_plain_views(eng.kv)))
        if small:
            eng.ws = eng.ws[:-1]
            with pytest.raises(tr.TRError) as e:
                eng.prefill(prompt[:140])
            assert e.value.status == tr.TR_ECAPACITY
    for i, (a, b) in enumerate(zip(*caches)):
        a, b = a.float(), b.float()
        if i < 2:
            # a bf16 value that sums of another order round the other way is 2^-8 off; two layers carry a few of them on
            assert float((a - b).norm() / a.norm()) < 4e-3 and float((a - b).abs().max()) < 6e-2 * float(a.abs().max())
        else:
            # a row on its own: each of the five bf16 roundings on the way may fall the other way, 5 x 2^-8 (measured 8e-3)
            a, b = a[:, :, :sum(lens)], b[:, :, :sum(lens)]
            err = (a - b).abs().amax(dim=(1, 3)) / a.abs().amax(dim=(1, 3))
            say("largest difference of a row", float(err.max()))
            assert float(err.max()) < 2e-2


def test_packed_prefill_appends_after_a_committed_prefix():
    """Two calls: 201 tokens, then 400 more on top (keep_cache).  The second call's wide pass starts at a
    non-zero committed length, so its rotary positions, cache rows and attention prefixes are all offset;
    the cache must equal the oracle's single causal prefill of all 600 tokens."""
    require_gpu()
    sh = synth.SHAPES["tiny_gqa_bf16"]
    w = synth.make_weights(sh, seed=4)
    wn = synth.weights_to_numpy(w)
    prompt = synth.zipf_prompt(sh.vocab, 601, seed=4).tolist()
    eng = tr.Engine(sh, to_gpu(w), synth.tree15(), k=K, capacity=720)
    assert eng.model.packed and eng.kv.tiled
    eng.prefill(prompt[:201])                      # commits 200, the 201st becomes the root and is dropped here
    eng.prefill(prompt[200:], keep_cache=True)     # commits tokens 200 .. 599
    torch.cuda.synchronize()
    n = 600
    assert int(eng.kv.d_len.item()) == n and eng.kv.c.len_bound == n
    cfg = oracle_cfg(sh)
    kv = O.KVCache(cfg, 720)
    O.prefill(cfg, wn, kv, prompt[:n])
    _cache_against_oracle(eng, kv, n)


def test_pack_weight_rope_interleaves_rows():
    """y = x W^T through a matrix packed with tr_pack_weight_rope comes out with output feature
    h*hd + 2j + b holding what feature h*hd + j + b*hd/2 holds with the plain packing."""
    require_gpu()
    n, K_, O_, hd = 33, 256, 512, 128
    x = synth.normal_tensor((n, K_), 1.0, seed=4, dtype=torch.bfloat16)
    wt = synth.uniform_tensor((O_, K_), float(np.sqrt(3.0 / K_)), seed=6, tensor_id=3, dtype=torch.bfloat16)
    ctx = tr.Context(16, 8, [-1], [-1], 1)
    ws = torch.empty(((n + 15) // 16 * 16 * K_ * 2 + 512 + n * O_ * 4 + 512), dtype=torch.uint8, device="cuda")
    y0 = torch.zeros(n, O_, dtype=torch.float32, device="cuda")
    y1 = torch.zeros_like(y0)
    ctx.op_linear(x.cuda(), tr.pack_weight(wt.cuda()), y0, ws, packed=True, splits=1)
    ctx.op_linear(x.cuda(), tr.pack_weight(wt.cuda(), rope_head_dim=hd), y1, ws, packed=True, splits=1)
    o = np.arange(O_)
    src = (o // hd) * hd + (o % hd) // 2 + ((o % hd) % 2) * (hd // 2)
    assert np.array_equal(y1.cpu().numpy(), y0.cpu().numpy()[:, src])
    with pytest.raises(tr.TRError):
        tr.pack_weight(wt.cuda(), rope_head_dim=96)            # 512 is not a multiple of 96


def test_capacity_is_checked_on_the_host():
    require_gpu()
    sh = synth.SHAPES["tiny"]
    w = synth.make_weights(sh, seed=2)
    tmpl = synth.tree15()
    eng = tr.Engine(sh, to_gpu(w), tmpl, k=K, capacity=64)
    assert eng.kv.capacity == 64
    with pytest.raises(tr.TRError) as e:
        eng.prefill(list(range(80)))
    assert e.value.status == tr.TR_ECAPACITY
    eng.prefill(list(range(55)))
    with pytest.raises(tr.TRError) as e:
        eng.step()                                            # 54 + 15 > 64
    assert e.value.status == tr.TR_ECAPACITY


@pytest.mark.parametrize("tmpl_name,H,Hkv,L,tiled", [("tree80", 32, 32, 1024, True), ("tree80", 8, 2, 1000, True),
                                                     ("tree81", 4, 4, 37, True), ("wide128", 4, 1, 300, True),
                                                     ("single", 8, 8, 513, True), ("tree15", 4, 4, 0, True),
                                                     ("tree80", 4, 2, 200, False),
                                                     # grouped-query shapes: the 70B head layout at its prompt
                                                     # length (two heads per workgroup), an odd group (one head
                                                     # per workgroup), six node tiles with shared heads, one node
                                                     ("tree80", 64, 8, 4096, True), ("tree80", 6, 2, 150, True),
                                                     ("prefix96", 8, 4, 70, True), ("single", 16, 2, 777, True)])
def test_tree_attention_matches_per_path_attention(tmpl_name, H, Hkv, L, tiled):
    """One layer of tree attention at the microbenchmark shape (32 heads x 128, prefix 1024, 80
    nodes, N(0,1) values) and smaller ones: every node must equal plain softmax attention over
    (prefix, its root-to-node path) computed by the oracle in float64."""
    require_gpu()
    say("tree attention", tmpl_name, H, Hkv, L, tiled)
    t = synth.prefix_template(int(tmpl_name[6:])) if tmpl_name.startswith("prefix") else synth.TEMPLATES[tmpl_name]()
    tree = O.make_tree(t.parent, t.rank, K)
    n, hd = t.n_nodes, 128
    sh = synth.ModelShape("att", 1, H * hd, H, Hkv, hd, 64, 64, "bf16")
    kv = tr.KVDesc(sh, capacity=L + n + 5, tiled=tiled)
    kv.reset(L)
    q = synth.normal_tensor((n, H, hd), 1.0, seed=1, dtype=torch.bfloat16)
    kp = synth.normal_tensor((1, Hkv, kv.capacity, hd), 1.0, seed=2, dtype=torch.bfloat16)
    vp = synth.normal_tensor((1, Hkv, kv.capacity, hd), 1.0, seed=3, dtype=torch.bfloat16)
    kv_fill(kv, kp.cuda(), vp.cuda())
    ctx = tr.Context(64, K, t.parent, t.rank, t.n_layers)
    out = torch.zeros(n, H, hd, dtype=torch.bfloat16, device="cuda")
    ws = torch.empty(16 * 128 * H * (2 + hd) * 4 + 4096, dtype=torch.uint8, device="cuda")
    ctx.op_tree_attention(kv, 0, H, q.cuda(), out, ws)
    got = out.float().cpu().numpy()
    qn = q.double().numpy()
    kn = kp[0].double().numpy().transpose(1, 0, 2)             # [cap, Hkv, hd]
    vn = vp[0].double().numpy().transpose(1, 0, 2)
    worst = 0.0
    for i in range(n):
        idx = list(range(L)) + [L + j for j in tree.paths[i]]
        ref = O._attend(qn[i], kn[idx], vn[idx], H // Hkv)
        err = np.abs(got[i] - ref).max()
        worst = max(worst, err / np.abs(ref).max())
        assert err <= 2e-2 * np.abs(ref).max(), (i, err)
    say("worst relative error", worst)


@pytest.mark.parametrize("tmpl_name,H,Hkv,L,slack", [
    # shares of an even and an odd number of tiles, the last step full, of one tile, partly tree, past the end; one to twelve waves
    ("tree80", 16, 16, 7900, 0), ("tree80", 40, 40, 2831, 0), ("tree81", 40, 40, 4432, 0), ("wide128", 64, 8, 5000, 0),
    ("prefix33", 40, 40, 2870, 0), ("prefix49", 40, 40, 2990, 0), ("prefix17", 64, 8, 3900, 0), ("prefix96", 64, 8, 3850, 0),
    ("tree80", 64, 8, 3800, 0), ("wide128", 64, 8, 5333, 0), ("prefix16", 10, 2, 7700, 0), ("prefix97", 40, 40, 4400, 0),
    # one share, no merge
    ("prefix66", 256, 256, 900, 0), ("wide128", 136, 136, 1160, 0),
    # the host's bound of the length is an estimate: above and (a step that reads more than it promised) below the true one
    ("tree80", 40, 40, 2900, 300), ("tree80", 40, 40, 2900, -64), ("prefix40", 40, 40, 2960, -64), ("prefix16", 10, 2, 7800, -96),
    ("tree80", 64, 8, 3900, 64), ("tree80", 64, 8, 3900, -64), ("wide128", 64, 8, 5100, -64), ("prefix66", 256, 256, 900, -40),
    # so far above that shares have one tile, or none, of what they asked for ahead
    ("tree80", 40, 40, 450, 2500), ("tree80", 40, 40, 10, 2900), ("wide128", 64, 8, 0, 5000), ("prefix40", 40, 40, 33, 2900), ("tree80", 64, 8, 100, 3800)])
def test_tree_attention_long_shares(tmpl_name, H, Hkv, L, slack):
    """The split form for long key shares at the edges of its steps, against softmax attention in float64.  bf16 results
    (2^-8 relative) of half-precision partial results (2^-11) and bf16 probabilities (2^-8 each, averaged): 1e-2 of the
    row's largest value."""
    require_gpu()
    say("tree attention, long shares", tmpl_name, H, Hkv, L, slack)
    t = synth.prefix_template(int(tmpl_name[6:])) if tmpl_name.startswith("prefix") else synth.TEMPLATES[tmpl_name]()
    tree = O.make_tree(t.parent, t.rank, K)
    n, hd = t.n_nodes, 128
    assert tr.plan_attention_form(H, Hkv, n, L + slack + n) == "long_shares"
    sh = synth.ModelShape("att", 1, H * hd, H, Hkv, hd, 64, 64, "bf16")
    kv = tr.KVDesc(sh, capacity=L + max(slack, 0) + n + 20)
    kv.reset(L)
    kv.c.len_bound = L + slack
    q = synth.normal_tensor((n, H, hd), 1.0, seed=1, dtype=torch.bfloat16)
    kp = synth.normal_tensor((1, Hkv, kv.capacity, hd), 1.0, seed=2, dtype=torch.bfloat16)
    vp = synth.normal_tensor((1, Hkv, kv.capacity, hd), 1.0, seed=3, dtype=torch.bfloat16)
    kv_fill(kv, kp.cuda(), vp.cuda())
    ctx = tr.Context(64, K, t.parent, t.rank, t.n_layers)
    out = torch.zeros(n, H, hd, dtype=torch.bfloat16, device="cuda")
    ws = torch.empty(16 * 128 * H * (2 + hd) * 4 + 4096, dtype=torch.uint8, device="cuda")
    ctx.op_tree_attention(kv, 0, H, q.cuda(), out, ws)
    seen = torch.zeros(n, L + n, dtype=torch.bool)
    seen[:, :L] = True
    for i in range(n):
        seen[i, [L + j for j in tree.paths[i]]] = True
    for h in range(0, H, max(1, H // 8)):
        g = h // (H // Hkv)
        s = q[:, h].double() @ kp[0, g, :L + n].double().T / hd ** 0.5
        ref = torch.softmax(s.masked_fill(~seen, -float("inf")), -1) @ vp[0, g, :L + n].double()
        err = (out[:, h].cpu().double() - ref).abs().amax(1) / ref.abs().amax(1)
        assert err.max() <= 1e-2, (h, err.max())
    ctx.close()


@pytest.mark.parametrize("tmpl_name,H,Hkv,L", [("tree80", 32, 32, 3900), ("wide128", 64, 8, 5000), ("prefix48", 64, 8, 3900),
                                               ("prefix24", 48, 16, 2500), ("prefix33", 40, 40, 2900), ("tree80", 64, 8, 3900)])
def test_tree_attention_long_shares_lose_no_precision(tmpl_name, H, Hkv, L):
    """All errors of the form for long key shares together, against float64, are those of the form for short ones (which blocks off 16
    bytes take): both move the running maximum after 32 keys, and only tiles with tree nodes round their exponents otherwise."""
    require_gpu()
    say("tree attention, precision", tmpl_name, H, Hkv, L)
    t = synth.prefix_template(int(tmpl_name[6:])) if tmpl_name.startswith("prefix") else synth.TEMPLATES[tmpl_name]()
    tree = O.make_tree(t.parent, t.rank, K)
    n, hd = t.n_nodes, 128
    assert tr.plan_attention_form(H, Hkv, n, L + n) == "long_shares"
    kv = tr.KVDesc(synth.ModelShape("att", 1, H * hd, H, Hkv, hd, 64, 64, "bf16"), capacity=L + n)
    kv.reset(L)
    q = synth.normal_tensor((n, H, hd), 1.0, seed=1, dtype=torch.bfloat16).cuda()
    kp = synth.normal_tensor((1, Hkv, kv.capacity, hd), 1.0, seed=2, dtype=torch.bfloat16).cuda()
    vp = synth.normal_tensor((1, Hkv, kv.capacity, hd), 1.0, seed=3, dtype=torch.bfloat16).cuda()
    kv_fill(kv, kp, vp)
    ctx = tr.Context(64, K, t.parent, t.rank, t.n_layers)
    ws = torch.empty(16 * 128 * H * (2 + hd) * 4 + 4096, dtype=torch.uint8, device="cuda")
    seen = torch.zeros(n, L + n, dtype=torch.bool)
    seen[:, :L] = True
    for i in range(n):
        seen[i, [L + j for j in tree.paths[i]]] = True
    ref = torch.empty(n, H, hd, dtype=torch.float64, device="cuda")
    for h in range(H):
        g = h // (H // Hkv)
        s = q[:, h].double() @ kp[0, g, :L + n].double().T / hd ** 0.5
        ref[:, h] = torch.softmax(s.masked_fill(~seen.cuda(), -float("inf")), -1) @ vp[0, g, :L + n].double()
    errs = []
    for off in (False, True):
        if off:
            kv.k, kv.v = _off_16(kv.k), _off_16(kv.v)
            kv.c.k, kv.c.v = kv.k.data_ptr(), kv.v.data_ptr()
        out = torch.zeros(n, H, hd, dtype=torch.bfloat16, device="cuda")
        ctx.op_tree_attention(kv, 0, H, q, out, ws)
        errs.append(float((out.double() - ref).norm() / ref.norm()))
    say("relative error, long form and short", errs)
    assert errs[0] <= 1.001 * errs[1]
    ctx.close()


@pytest.mark.parametrize("dtype,hd", [("f32", 64), ("bf16", 128), ("f32", 30)])
def test_generic_attention_ignores_what_a_node_does_not_see(dtype, hd):
    """Shape-generic attention: a tree node whose value vector is not finite reaches its descendants and itself, and
    leaves every other row what it is with a finite one."""
    require_gpu()
    say("generic attention, non-finite sibling", dtype, hd)
    t = synth.tree15()
    tree = O.make_tree(t.parent, t.rank, K)
    n, H, Hkv, L = t.n_nodes, 4, 2, 260
    sh = synth.ModelShape("att", 1, H * hd, H, Hkv, hd, 64, 64, dtype)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    q = synth.normal_tensor((n, H, hd), 1.0, seed=1, dtype=dt).cuda()
    kp = synth.normal_tensor((1, Hkv, L + n + 5, hd), 1.0, seed=2, dtype=dt)
    vp = synth.normal_tensor((1, Hkv, L + n + 5, hd), 1.0, seed=3, dtype=dt)
    ctx = tr.Context(64, K, t.parent, t.rank, t.n_layers)
    outs = []
    bad = {2: float("nan"), 5: float("inf")}
    for values in ({}, bad):
        kv = tr.KVDesc(sh, capacity=L + n + 5, tiled=False)
        kv.reset(L)
        pad = kv.capacity - kp.shape[2]
        k, v = (torch.nn.functional.pad(a, (0, 0, 0, pad)) for a in (kp, vp))
        for node, x in values.items():
            v[0, :, L + node, :] = x
        kv_fill(kv, k.cuda(), v.cuda())
        out = torch.zeros(n, H, hd, dtype=dt, device="cuda")
        ws = torch.empty(16 * 128 * H * (2 + hd) * 4 + 4096, dtype=torch.uint8, device="cuda")
        ctx.op_tree_attention(kv, 0, H, q, out, ws)
        outs.append(out.cpu())
    for i in range(n):
        if set(tree.paths[i]) & set(bad):
            assert not outs[1][i].isfinite().any(), i
        else:
            assert torch.equal(outs[0][i], outs[1][i]), i
    ctx.close()


@pytest.mark.parametrize("tmpl_name,H,Hkv,L", [("single", 16, 2, 0), ("single", 16, 2, 40), ("single", 64, 8, 800), ("prefix3", 64, 8, 3001),
                                               ("prefix20", 8, 8, 900), ("prefix32", 4, 4, 1201),               # one tile of 32 rows
                                               ("prefix8", 64, 8, 1500), ("prefix40", 2, 2, 7190),              # two
                                               ("prefix12", 64, 8, 3100), ("prefix24", 16, 4, 8200),            # three
                                               ("tree15", 64, 8, 3333), ("prefix16", 8, 1, 5001),               # four
                                               # what the rule gives the form: 32, 64, 96 and 128 rows, one share and several,
                                               # groups of one, two and such that rows do not fall on their bounds by shifts
                                               ("single", 16, 2, 32), ("prefix10", 12, 4, 97), ("prefix3", 14, 2, 219),
                                               ("prefix32", 8, 8, 5170), ("prefix16", 16, 8, 5190), ("prefix10", 12, 4, 1500),
                                               ("prefix4", 14, 2, 1100), ("prefix5", 56, 8, 5120), ("prefix21", 6, 2, 5100),
                                               ("prefix13", 28, 4, 8180), ("prefix18", 28, 4, 8193), ("prefix42", 24, 8, 8200),
                                               ("prefix8", 64, 8, 2000), ("prefix16", 64, 8, 4001)])
def test_few_rows_attention(tmpl_name, H, Hkv, L):
    """The form for few (node, head) rows per K/V head, every row-tile count of it: sequences shorter than its first step,
    one key share and many, last tiles partly tree, partly past the end.  Sizes around its use that the rule leaves to the
    other forms stay in the list; those it takes are asserted."""
    n = (synth.prefix_template(int(tmpl_name[6:])) if tmpl_name.startswith("prefix") else synth.TEMPLATES[tmpl_name]()).n_nodes
    left = {("single", 16, 2, 0), ("prefix20", 8, 8, 900), ("prefix32", 4, 4, 1201), ("prefix8", 64, 8, 1500),
            ("prefix40", 2, 2, 7190), ("prefix16", 8, 1, 5001)}
    assert (tr.plan_attention(H, Hkv, n, L + n)[1] < 0) == ((tmpl_name, H, Hkv, L) not in left)
    test_tree_attention_matches_per_path_attention(tmpl_name, H, Hkv, L, True)


@pytest.mark.parametrize("tmpl_name,H,Hkv,L", [("single", 16, 2, 40), ("prefix3", 64, 8, 150), ("prefix3", 64, 8, 3001)])
def test_few_rows_attention_without_a_finite_score(tmpl_name, H, Hkv, L):
    """A row whose query is not a number, or whose scores are all -inf, has no softmax: its result is NaN with one key
    share and with several, and the other rows are what they are without it."""
    require_gpu()
    say("few rows, no finite score", tmpl_name, H, Hkv, L)
    t = synth.prefix_template(int(tmpl_name[6:])) if tmpl_name.startswith("prefix") else synth.TEMPLATES[tmpl_name]()
    n = t.n_nodes
    kv = tr.KVDesc(synth.ModelShape("att", 1, H * 128, H, Hkv, 128, 64, 64, "bf16"), capacity=L + n)
    kv.reset(L)
    kp = synth.normal_tensor((1, Hkv, kv.capacity, 128), 1.0, seed=2, dtype=torch.bfloat16)
    vp = synth.normal_tensor((1, Hkv, kv.capacity, 128), 1.0, seed=3, dtype=torch.bfloat16)
    kp[0, 0, :L + n, 5] = -float("inf")        # K/V head 0: -inf wherever the query's feature 5 is positive
    kv_fill(kv, kp.cuda(), vp.cuda())
    ctx = tr.Context(64, K, t.parent, t.rank, t.n_layers)
    ws = torch.empty(16 * 128 * H * 130 * 4 + 4096, dtype=torch.uint8, device="cuda")
    q = synth.normal_tensor((n, H, 128), 1.0, seed=1, dtype=torch.bfloat16)
    q[:, :, 5] = 1.0
    outs = []
    for bad in (False, True):
        if bad:
            q[n - 1, H - 1, 17] = float("nan")
        out = torch.zeros(n, H, 128, dtype=torch.bfloat16, device="cuda")
        ctx.op_tree_attention(kv, 0, H, q.cuda(), out, ws)
        outs.append(out.cpu())
    G = H // Hkv
    assert outs[0][:, :G].isnan().all() and outs[0][:, G:].isfinite().all()
    assert outs[1][n - 1, H - 1].isnan().all()
    outs[1][n - 1, H - 1] = outs[0][n - 1, H - 1]
    assert torch.equal(outs[0][:, G:], outs[1][:, G:])
    ctx.close()


@pytest.mark.parametrize("n,K_,O_,splits", [(80, 4096, 4096, 2), (80, 11008, 4096, 2), (81, 4096, 1024, 4),
                                            (1, 4096, 512, 1), (128, 512, 2048, 1), (16, 256, 64, 1),
                                            (80, 1024, 32000, 1), (80, 4096, 12288, 1), (37, 96, 32, 3),
                                            # above 128 rows: the prompt-ingestion kernel in each of its shapes
                                            (129, 64, 32, 1), (250, 4096, 4096, 4), (256, 736, 2080, 1),
                                            (300, 256, 18432, 1), (511, 4096, 4608, 4), (512, 11008, 4096, 4),
                                            (401, 4096, 1024, 4), (300, 2240, 96, 3)])
def test_linear_bf16_packed_matches_oracle_matmul(n, K_, O_, splits):
    """The projection kernel alone (packed weights, MFMA) against a float64 matrix product of the
    same bf16 values; also checks the repack kernel, since a misplaced element would show here.
    Row counts above 128 reach the prompt-ingestion kernel, whose launcher picks the workgroup shape (8 or 16 row
    tiles x 8, 12 or 16 out-tiles) and the K-splits from a cost model: the cases cover one and several row blocks,
    ragged out-tile groups (2080 features), an odd number of k-steps (736) and K-split shares that leave a shorter
    last share (2240 in-features); test_wide_projection_edges has every shape."""
    require_gpu()
    say("linear packed", n, K_, O_, splits)
    x = synth.normal_tensor((n, K_), 1.0, seed=n + K_, dtype=torch.bfloat16)
    w = synth.uniform_tensor((O_, K_), float(np.sqrt(3.0 / K_)), seed=5, tensor_id=O_, dtype=torch.bfloat16)
    ctx = tr.Context(16, 8, [-1], [-1], 1)
    y = torch.zeros(n, O_, dtype=torch.float32, device="cuda")
    ws = torch.empty(((n + 15) // 16 * 16 * K_ * 2 + 512 + splits * n * O_ * 4 + 512), dtype=torch.uint8, device="cuda")
    wp = tr.pack_weight(w.cuda())
    ctx.op_linear(x.cuda(), wp, y, ws, packed=True, splits=splits)
    ref = x.double().numpy() @ w.double().numpy().T
    err = np.abs(y.cpu().numpy() - ref).max()
    say("max err", err)
    assert err < 2e-5 * np.sqrt(K_)                           # fp32 accumulation of K products of O(1/sqrt(K))


@pytest.mark.parametrize("n,K_,O_,splits", [# workgroups of 8 x 8 tiles: fewer k-steps than ring slots, an odd number
                                            (129, 64, 64, 1), (135, 96, 256, 1), (200, 160, 64, 1), (257, 1120, 8224, 2),
                                            (512, 4096, 4096, 4), (511, 4096, 4640, 3),  # 8 x 8, split over k and not
                                            (511, 4096, 12288, 1), (250, 1056, 24576, 1),  # 8 x 12
                                            (500, 96, 12320, 1),                  # 16 x 8; one ragged row block, split
                                            (129, 1056, 24576, 1), (145, 3072, 6144, 4),
                                            (505, 1056, 16416, 1), (385, 96, 20512, 1),                        # 16 x 12
                                            (505, 736, 28704, 1), (400, 224, 32000, 1), (512, 64, 28704, 1)])  # 16 x 16
def test_wide_projection_edges(n, K_, O_, splits):
    """Prompt-ingestion projection in every workgroup shape its launcher has: k ranges shorter than, equal to and past
    the LDS ring, odd and even numbers of k-steps, last row block and last out-tile group partly empty."""
    require_gpu()
    say("wide projection", n, K_, O_, splits)
    x = synth.normal_tensor((n, K_), 1.0, seed=n + K_, dtype=torch.bfloat16).cuda()
    w = synth.uniform_tensor((O_, K_), float(np.sqrt(3.0 / K_)), seed=9, tensor_id=O_, dtype=torch.bfloat16).cuda()
    ctx = tr.Context(16, 8, [-1], [-1], 1)
    y = torch.full((n, O_), float("nan"), dtype=torch.float32, device="cuda")
    ws = torch.empty(((n + 15) // 16 * 16 * K_ * 2 + 512 + splits * n * O_ * 4 + 512), dtype=torch.uint8, device="cuda")
    ctx.op_linear(x, tr.pack_weight(w), y, ws, packed=True, splits=splits)
    ref = x.double() @ w.double().T
    # K products of O(1/sqrt(K)), each rounded to 2^-24 of the running sum on its way into it
    assert float((y.double() - ref).abs().max()) < 2e-5 * np.sqrt(K_)
    ctx.close()


def _off_16(x):
    """The same values in memory that starts 8 bytes behind a multiple of 16."""
    buf = torch.empty(x.numel() + 8, dtype=x.dtype, device=x.device)
    y = buf[4:4 + x.numel()].view(x.shape).copy_(x)
    assert y.data_ptr() % 16 == 8
    return y


@pytest.mark.parametrize("what", ["weights", "cache", "workspace"])
def test_prefill_from_blocks_off_16_bytes(what):
    """Prompt ingestion with weights, a cache or a workspace that does not start on 16 bytes (a caller's own arena): the
    kernels that load straight into LDS are not for them; the cache comes out as from aligned ones."""
    require_gpu()
    say("prefill off 16 bytes", what)
    sh = synth.SHAPES["tiny_gqa_bf16"]
    w = to_gpu(synth.make_weights(sh, seed=6))
    prompt = synth.zipf_prompt(sh.vocab, 301, seed=6).tolist()
    caches = []
    for off in (False, True):
        eng = tr.Engine(sh, w, synth.tree15(), k=K, capacity=352)
        if off and what == "workspace":
            eng.ws = torch.cat([eng.ws, eng.ws[:16]])[8:]
            assert eng.ws.data_ptr() % 16 == 8
        elif off and what == "cache":
            eng.kv.k, eng.kv.v = _off_16(eng.kv.k), _off_16(eng.kv.v)
            eng.kv.c.k, eng.kv.c.v = eng.kv.k.data_ptr(), eng.kv.v.data_ptr()
        elif off:
            keep = [_off_16(lw["w_gate"]) for lw in eng.model.weights["layers"]]
            for l, x in enumerate(keep):
                eng.model._layers[l].w_gate = x.data_ptr()
        eng.prefill(prompt)
        torch.cuda.synchronize()
        assert int(eng.kv.d_len.item()) == 300
        caches.append([x[:, :, :300].float() for x in kv_plain_views(eng.kv)])
    for a, b in zip(*caches):
        # per row; two bf16 forwards with their sums in another order
        err = (a - b).abs().amax(dim=(1, 3)) / a.abs().amax(dim=(1, 3))
        assert float(err.max()) < 2e-2


def _uniform(gen, out_f, in_f, std=1.0):
    s = std * (3.0 / in_f) ** 0.5
    return torch.empty(out_f, in_f, dtype=torch.bfloat16, device="cuda").uniform_(-s, s, generator=gen)


def _feed_forward_step(shape, n, seed, moved=(), counted=False, past=None, **given):
    """One step of one layer whose attention adds nothing (wo = 0); `given` replaces weights, `moved` names those that start off 16
    bytes, `past` are the keys and values of the cache (zeros).  With `counted`, eng.launches holds how often the step launched each kind
    of kernel.  Returns the engine behind the step, its weights and the embeddings of its tokens in float64."""
    d, F, gen = shape.d_model, shape.d_ffn, torch.Generator("cuda").manual_seed(seed)
    hq, hk = shape.n_heads * shape.head_dim, shape.n_kv_heads * shape.head_dim
    ones = torch.ones(d, dtype=torch.bfloat16, device="cuda")
    w = {"embed": _uniform(gen, shape.vocab, d, d ** 0.5), "lm_head": _uniform(gen, shape.vocab, d), "final_norm": ones, "layers": [
        {"attn_norm": ones, "ffn_norm": ones, "wq": _uniform(gen, hq, d), "wk": _uniform(gen, hk, d), "wv": _uniform(gen, hk, d),
         "wo": torch.zeros(d, hq, dtype=torch.bfloat16, device="cuda"), "w_gate": _uniform(gen, F, d), "w_up": _uniform(gen, F, d),
         "w_down": _uniform(gen, d, F)}]}
    for name, x in given.items():
        (w if name in w else w["layers"][0])[name] = x
    eng = tr.Engine(shape, w, synth.prefix_template(n) if n > 1 else synth.single(), k=K, capacity=320)
    eng.moved = {m: _off_16(eng.model.weights[m] if m == "lm_head" else eng.model.weights["layers"][0][m]) for m in moved}
    for m, x in eng.moved.items():
        setattr(eng.model.c if m == "lm_head" else eng.model._layers[0], m, x.data_ptr())
    eng.kv.reset(150)
    if past is not None:
        kv_fill(eng.kv, *past, k_interleaved=True)
    eng.ctx.matrix_load(np.random.default_rng(n).integers(0, shape.vocab, (shape.vocab, K), dtype=np.int32))
    eng.root.fill_(7)
    if counted:
        eng.ctx.profile_enable(True)
    eng.step()
    torch.cuda.synchronize()
    if counted:
        eng.launches = {kind: launches for kind, (launches, _) in eng.ctx.profile_read().items()}
    return eng, w, w["embed"][eng.S.long()].double()


def _half_embedding(d, seed):
    """Tokens in the first half of the features, the other half left to what the layer writes there."""
    e = torch.zeros(d, d, dtype=torch.bfloat16, device="cuda")
    e[:, :d // 2].uniform_(-1.75, 1.75, generator=torch.Generator("cuda").manual_seed(seed))
    return e


def _stream_of(eng, xe):
    """The residual stream, rounded to bf16, from the logits of an identity LM head: they are it times one RMS scale a row, which the
    half that the layer does not write gives back."""
    first = xe[:, :xe.shape[1] // 2]
    scale = (eng.logits[:, :first.shape[1]].double() * first).sum(1) / (first * first).sum(1)
    return eng.logits.double() / scale[:, None], scale


@pytest.mark.parametrize("d,F,out_tiles,nodes", [
    # 201 workgroups each, the last one partly filled; an even and an odd number of k-steps, for the two groups of waves too
    (4096, 12832, 8, (65, 80, 81, 97, 128)), (5152, 12832, 8, (33, 48)), (4096, 25632, 16, (33, 49, 80, 113, 128)),
    (5152, 25632, 16, (17, 32, 97)), (4160, 9632, 6, (97, 112, 113, 128)), (4224, 9664, 6, (97, 128)),
    (4096, 12832, 0, (1, 16, 48, 49, 64)), (4096, 9632, 0, (80, 96))])           # the decode kernel's rows beside them
def test_step_projections_with_many_out_tiles(d, F, out_tiles, nodes):
    """Gate/up and SwiGLU in every form of the kernel that shares operands in LDS, feature by feature against float64: w_down adds
    features f, f + d / 2, .. with weights 1, -9/8, 10/8, .. to one feature of the residual stream.  Two bf16 roundings of 2^-8
    (the SwiGLU output, the stream) and float32 sums."""
    require_gpu()
    half = d // 2
    shape = synth.ModelShape("many", 1, d, 2, 1, 128, F, d, "bf16")
    f = torch.arange(F, device="cuda")
    w_down = torch.zeros(d, F, dtype=torch.bfloat16, device="cuda")
    w_down[half + f % half, f] = ((1 + (f // half) / 8) * (1 - 2 * (f // half % 2))).to(torch.bfloat16)
    eye, embed = torch.eye(d, dtype=torch.bfloat16, device="cuda"), _half_embedding(d, F)
    for n in nodes:
        say("step projections", d, F, n)
        p, _, splits, kernel = tr.plan_step_projection("gate_up", n, d, F)
        assert (2 * p * kernel, splits) == (out_tiles, 1)
        eng, w, xe = _feed_forward_step(shape, n, 4, embed=embed, w_down=w_down, lm_head=eye)
        got, _ = _stream_of(eng, xe)
        a = xe / (xe.square().mean(1, keepdim=True) + shape.rms_eps).sqrt()
        lw = w["layers"][0]
        gate, up = a @ lw["w_gate"].double().T, a @ lw["w_up"].double().T
        h = gate * torch.sigmoid(gate) * up
        ref, size = h @ w_down[half:].double().T, h.abs() @ w_down[half:].double().abs().T
        over = (got[:, half:] - ref).abs() / (2.0 ** -8 * (size + ref.abs()) + 1e-4)
        assert float(over.max()) < 1.01, (n, float(over.max()))


@pytest.mark.parametrize("d,F,shared,nodes", [(6432, 16416, True, (81, 96, 97, 128)), (6432, 21792, True, (113, 128)),
                                              (6432, 16416, False, (1, 64, 80)), (6432, 16256, False, (96,))])
def test_step_projections_in_shares_of_k(d, F, shared, nodes):
    """Down in four shares of k, the last one shorter, output by output against float64 of the rounded SwiGLU output: a value of that may
    round the other way, 2^-8 of some of the F terms, and the stream is rounded to bf16.  One k-step left out is 0.04 of a standard
    deviation on average."""
    require_gpu()
    shape = synth.ModelShape("shares", 1, d, 2, 1, 128, F, d, "bf16")
    eye = torch.eye(d, dtype=torch.bfloat16, device="cuda")
    for n in nodes:
        say("step projections in shares", d, F, n)
        assert tr.plan_step_projection("o_down", n, F, d)[3] == int(shared)
        eng, w, xe = _feed_forward_step(shape, n, 5, lm_head=eye)
        a = xe / (xe.square().mean(1, keepdim=True) + shape.rms_eps).sqrt()
        lw = w["layers"][0]
        gate, up = a @ lw["w_gate"].double().T, a @ lw["w_up"].double().T
        add = (gate * torch.sigmoid(gate) * up).to(torch.bfloat16).double() @ lw["w_down"].double().T
        ref = xe + add
        got = eng.logits.double()
        got = got * ((ref * ref).sum(1) / (got * ref).sum(1))[:, None]     # the row's RMS scale
        over = (got - ref).abs() / (2.0 ** -8 * ref.abs() + 0.02 * add.std())
        assert float(over.max()) < 1.01, (n, float(over.max()))


@pytest.mark.parametrize("d,F,groups", [(3232, 256, 202), (4064, 512, 254), (4096, 256, 256), (6400, 512, 200), (8192, 256, 256)])
def test_projections_that_update_the_residual_stream(d, F, groups):
    """o and down of one and two row tiles, which add to the residual stream in their own epilogue: the stream behind them output by
    output as in test_step_projections_in_shares_of_k, and the RMS scale that the sums of squares of all workgroups give (the rounding of
    d independent outputs leaves 2^-9 / sqrt(d) of it).  Gains are powers of two, so that they round nothing."""
    require_gpu()
    shape = synth.ModelShape("resid", 1, d, 2, 1, 128, F, d, "bf16")
    eye = torch.eye(d, dtype=torch.bfloat16, device="cuda")
    gen = torch.Generator("cuda").manual_seed(d)
    gains = [(2.0 ** torch.randint(-1, 2, (d,), device="cuda", generator=gen)).to(torch.bfloat16) for _ in range(2)]
    taken = 0
    for n in (1, 2, 15, 16, 17, 31, 32, 33):
        say("residual epilogue", d, F, n)
        plans = [tr.plan_step_projection("o_down", n, in_f, d) for in_f in (256, F)]       # o and down
        fused = [200 <= g <= 256 and (splits, kernel) == (1, 0) and n <= 32 for _, g, splits, kernel in plans]
        taken += all(fused) and plans[1][1] == groups
        eng, w, xe = _feed_forward_step(shape, n, 6, counted=True, lm_head=eye, ffn_norm=gains[0], final_norm=gains[1])
        assert eng.launches.get("residual_norm", 0) == 2 - sum(fused), (n, eng.launches)
        a = xe * gains[0].double() / (xe.square().mean(1, keepdim=True) + shape.rms_eps).sqrt()
        lw = w["layers"][0]
        gate, up = a @ lw["w_gate"].double().T, a @ lw["w_up"].double().T
        add = (gate * torch.sigmoid(gate) * up).to(torch.bfloat16).double() @ lw["w_down"].double().T
        ref = xe + add
        got = eng.logits.double() / gains[1].double()
        scale = (got * ref).sum(1) / (ref * ref).sum(1)
        over = (got / scale[:, None] - ref).abs() / (2.0 ** -8 * ref.abs() + 0.02 * add.std())
        assert float(over.max()) < 1.01, (n, float(over.max()))
        assert float((scale * (ref.square().mean(1) + shape.rms_eps).sqrt() - 1).abs().max()) < 1e-3, n
    assert taken >= 4


@pytest.mark.parametrize("d,heads,kv_heads,nodes,shares", [
    (8192, 64, 8, (32, 33, 80, 128), (33, 80, 128)), (8192, 40, 8, (49, 64, 65), (49, 64, 65)),
    (5120, 40, 40, (80, 96, 97, 128), (97, 128)), (5152, 80, 16, (81, 97, 113), (97, 113))])
def test_qkv_in_shares_of_k(d, heads, kv_heads, nodes, shares):
    """Q/K/V in two, three and four shares of k, and the rows where it stays whole or a matrix off 16 bytes keeps it whole: keys and values
    of all nodes against float64 (one bf16 rounding of at most 2^-9 and float32 sums), the queries through what the attention makes of
    them.  It runs behind 150 random positions with scores of standard deviation 3, and wo and the LM head hand its output on feature by
    feature, so that every 32 features of a row are compared with float64 behind queries, keys and values in bf16.  Probabilities, output and
    stream are rounded by up to 2^-9 each, the first against sum p |v|, up to four times the output: 6 * 2^-9.  The reference with the
    queries of one row, of one head or of a pair of a head's features left out has to be further away."""
    require_gpu()
    hq, P = heads * 128, 150
    shape = synth.ModelShape("qkv", 1, d, heads, kv_heads, 128, 256, d, "bf16")
    gen, eye = torch.Generator("cuda").manual_seed(3), torch.eye(d, dtype=torch.bfloat16, device="cuda")
    f = torch.arange(hq, device="cuda")
    wo = torch.zeros(d, hq, dtype=torch.bfloat16, device="cuda")            # more heads than features: features f and f + d meet
    wo[f % d, f] = ((1 + (f // d) / 8) * (1 - 2 * (f // d % 2))).to(torch.bfloat16)
    given = dict(wo=wo, lm_head=eye, embed=_uniform(gen, d, d, d ** 0.5 / 64), wq=_uniform(gen, hq, d, 3.0),
                 w_down=torch.zeros(d, 256, dtype=torch.bfloat16, device="cuda"))
    past = [torch.randn(1, kv_heads, 320, 128, device="cuda", generator=gen).to(torch.bfloat16) for _ in range(2)]
    for n in nodes:
        say("qkv in shares", d, heads, kv_heads, n)
        parent, depth, anc = synth.prefix_template(n).parent, np.zeros(n), np.eye(n, dtype=bool)
        for i in range(1, n):
            depth[i] = depth[parent[i]] + 1
            anc[i] |= anc[parent[i]]
        seen = torch.from_numpy(np.concatenate([np.ones((n, P), bool), anc], 1))
        angle = (P + torch.from_numpy(depth).cuda())[:, None] * 10000.0 ** (-torch.arange(64, device="cuda").double() / 64)
        cos, sin = angle.cos()[:, None], angle.sin()[:, None]

        def rotated(x):
            return torch.cat([x[..., :64] * cos - x[..., 64:] * sin, x[..., 64:] * cos + x[..., :64] * sin], -1)

        split = tr.plan_step_qkv(n, d, heads, kv_heads)[2] > 1
        assert split == (n in shares), n
        for moved, launches in (((), 1 + split), (("wq",), 1)):
            eng, w, xe = _feed_forward_step(shape, n, 9, moved=moved, counted=True, past=past, **given)
            assert eng.launches["qkv_proj"] == launches, n
            lw, a = w["layers"][0], xe / (xe.square().mean(1, keepdim=True) + shape.rms_eps).sqrt()
            q = rotated((a @ lw["wq"].double().T).view(n, heads, 128)).cpu()
            k = rotated((a @ lw["wk"].double().T).view(n, kv_heads, 128))
            v = (a @ lw["wv"].double().T).view(n, kv_heads, 128)
            kp, vp = kv_plain_views(eng.kv, k_interleaved=True)
            moved_rows = int(eng.kv.d_len.item()) - P                  # the accepted nodes lie there now
            for got, ref in ((kp, k), (vp, v)):
                got = got[0, :, P:P + n].permute(1, 0, 2).double()
                over = (got - ref).abs() / (2.0 ** -8 * ref.abs() + 1e-5)
                assert float(over[moved_rows:].max()) < 1.01 and float(over[0].max()) < 1.01, (n, float(over.max()))
            keys, values = (torch.cat([c[0, :, :P], x.permute(1, 0, 2).to(torch.bfloat16)], 1).double().cpu() for c, x in zip(past, (k, v)))
            got, xe, out = eng.logits.double().cpu(), xe.cpu(), wo.double().cpu()

            def worst(q):
                """Largest relative error of 32 features of a row, with these queries in the reference."""
                o = torch.empty(n, heads, 128, dtype=torch.float64)
                for h in range(heads):
                    s = (q[:, h].to(torch.bfloat16).double() @ keys[h * kv_heads // heads].T) / 128 ** 0.5
                    o[:, h] = torch.softmax(s.masked_fill(~seen, -np.inf), 1) @ values[h * kv_heads // heads]
                ref = xe + o.view(n, hq) @ out.T
                scale = (got * ref).sum(1) / (ref * ref).sum(1)
                err, size = ((x.view(n, -1, 32)).norm(dim=2) for x in (got / scale[:, None] - ref, ref))
                return float((err / size).max())

            error = worst(q)
            say("largest relative error of 32 features", error)
            assert error < 6 * 2.0 ** -9, (n, error)
            for rows, hs, feats in ((n - 1, slice(None), slice(None)), (slice(None), heads - 1, slice(None)), (slice(None), 0, [5, 69])):
                wrong = q.clone()
                wrong[rows, hs, feats] = 0
                assert worst(wrong) > 5e-2, (rows, hs, feats)          # the comparison tells


@pytest.mark.parametrize("d,vocab,out_tiles,nodes", [
    # 201 workgroups of 8 and of 16 out-tiles, the last one partly filled, and several rounds of both
    (4096, 25632, 8, (65, 80, 97, 128)), (5152, 25632, 8, (33, 48)), (4096, 76832, 8, (81, 128)), (4096, 51232, 16, (33, 49, 128)),
    (5152, 51232, 16, (17, 32, 80)), (4096, 102432, 16, (49, 128)), (4096, 25632, 0, (1, 64)), (4096, 51232, 0, (1, 32))])
def test_lm_head_of_many_out_tiles(d, vocab, out_tiles, nodes):
    """LM heads that share operands in LDS, logit by logit against float64 (at most 80 roundings on a product's way, each half an
    ulp of at most sum |a w|), and all errors together against the decode kernel's, which a matrix off 16 bytes takes: they are
    as small."""
    require_gpu()
    shape = synth.ModelShape("head", 1, d, 2, 1, 128, 64, vocab, "bf16")
    zero = torch.zeros(d, 64, dtype=torch.bfloat16, device="cuda")
    for n in nodes:
        say("LM head", d, vocab, n)
        p, _, splits, kernel = tr.plan_step_projection("lm_head", n, d, vocab)
        assert (p * kernel, splits) == (out_tiles, 1)
        errs = []
        for moved in ((), ("lm_head",)):
            eng, w, xe = _feed_forward_step(shape, n, 6, moved, w_down=zero)
            a = xe / (xe.square().mean(1, keepdim=True) + shape.rms_eps).sqrt()
            num = den = 0.0
            for lo in range(0, vocab, 16384):
                wt = w["lm_head"][lo:lo + 16384].double().T
                ref, size = a @ wt, a.abs() @ wt.abs()
                err = (eng.logits[:, lo:lo + 16384].double() - ref).abs()
                assert float((err / size).max()) < 80 * 2.0 ** -24, (n, lo)
                num, den = num + float(err.square().sum()), den + float(ref.square().sum())
            errs.append((num / den) ** 0.5)
            del eng, w
        say("relative error, this kernel and the decode kernel", errs)
        assert errs[0] <= 1.02 * errs[1]


@pytest.mark.parametrize("d,F,out_tiles,n", [(512, 1024, 0, 80), (512, 1056, 0, 5), (4096, 12832, 8, 80), (4096, 25632, 16, 49),
                                             (4096, 9632, 6, 113)])
def test_swiglu_over_the_range_of_the_gate(d, F, out_tiles, n):
    """silu(gate) * up, rounded once to bf16, for gates from -110 to 100 against float64, in the decode kernel and in every form of
    the one that shares operands in LDS.  Besides its rounding, 2^-8, a result carries what the float32 sums are off by: a chain of up to
    64 additions, each rounded to half an ulp of up to 110 for the gate (2.5e-4 in all) and of a few units for up (1e-5).
    Below -88.7 e^-gate is beyond float32 and the result 0."""
    require_gpu()
    say("swiglu over the gate's range", d, F, n)
    shape, half = synth.ModelShape("gates", 1, d, 2, 1, 128, F, d, "bf16"), d // 2
    gen = torch.Generator("cuda").manual_seed(F + n)
    want = -110.0 * torch.rand(F, device="cuda", generator=gen)          # mostly negative: a few large rows do not set the scale
    at = torch.rand(F, device="cuda", generator=gen)
    want = torch.where(at < 0.35, -87.9 + 0.8 * (at / 0.35 - 0.5), want) # where the quotient leaves the normal numbers
    want = torch.where(at > 0.98, 20 * torch.rand(F, device="cuda", generator=gen), want)
    want = torch.where(at > 0.997, 100.0, want)
    want[F - 16] = 100.0
    embed, w_gate = _half_embedding(d, F), _uniform(gen, F, d, 0.125)
    embed[:, 0] = 8.0                                                    # feature 0 alone sets a gate but for some 0.1
    w_gate[:, 0] = want * ((64 + (half - 1)) / d) ** 0.5 / 8.0
    sel = torch.randperm(F, generator=gen, device="cuda")[:half]
    sel[:16], sel[-16:] = torch.arange(16, device="cuda"), torch.arange(F - 16, F, device="cuda")
    w_down = torch.zeros(d, F, dtype=torch.bfloat16, device="cuda")
    w_down[half + torch.arange(half, device="cuda"), sel] = 1
    assert (2 * tr.plan_step_projection("gate_up", n, d, F)[0] if d > 512 else 0) == out_tiles
    eng, w, xe = _feed_forward_step(shape, n, 9, embed=embed, w_gate=w_gate, w_down=w_down,
                                    lm_head=torch.eye(d, dtype=torch.bfloat16, device="cuda"))
    got, scale = _stream_of(eng, xe)
    got = got[:, half:]
    a = xe / (xe.square().mean(1, keepdim=True) + shape.rms_eps).sqrt()
    gate, up = a @ w_gate[sel].double().T, a @ w["layers"][0]["w_up"][sel].double().T
    sig = torch.sigmoid(gate)
    ref = gate * sig * up
    sure = (gate > -88.6) & (ref.abs() * scale[:, None] > 2.0 ** -124)   # normal numbers all the way
    assert int(((gate < -87.4) & sure).sum()) > 50 and float(gate.max()) > 80
    bound = 2.0 ** -8 * ref.abs() + 2.5e-4 * (up * sig * (1 + gate * (1 - sig))).abs() + 1e-5 * (gate * sig).abs()
    err = ((got - ref).abs() / bound)[sure]
    say("largest error over its bound", float(err.max()))
    assert float(err.max()) < 1.01
    rest = ~sure
    assert bool((got[rest].abs() <= ref[rest].abs() * 1.01 + 2.0 ** -120).all())


def test_attention_and_linear_from_blocks_off_16_bytes():
    require_gpu()
    say("attention and linear off 16 bytes")
    sh = synth.ModelShape("att", 1, 64 * 128, 64, 8, 128, 64, 64, "bf16")
    t = synth.prefix_template(3)
    q = synth.normal_tensor((3, 64, 128), 1.0, seed=1, dtype=torch.bfloat16).cuda()
    ctx = tr.Context(64, K, t.parent, t.rank, t.n_layers)
    ws = torch.empty(16 * 128 * 64 * 130 * 4 + 4096, dtype=torch.uint8, device="cuda")
    kv = tr.KVDesc(sh, capacity=1504)
    kv.reset(1500)
    kv.k.copy_(synth.normal_tensor(tuple(kv.k.shape), 1.0, seed=2, dtype=torch.bfloat16))
    kv.v.copy_(synth.normal_tensor(tuple(kv.v.shape), 1.0, seed=3, dtype=torch.bfloat16))
    assert tr.plan_attention(64, 8, 3, 1503)[1] < 0
    outs = []
    for off in (False, True):
        if off:
            kv.k, kv.v = _off_16(kv.k), _off_16(kv.v)
            kv.c.k, kv.c.v = kv.k.data_ptr(), kv.v.data_ptr()
        out = torch.zeros(3, 64, 128, dtype=torch.bfloat16, device="cuda")
        ctx.op_tree_attention(kv, 0, 64, q, out, ws)
        outs.append(out.float())
    assert float((outs[0] - outs[1]).abs().max()) < 2e-2 * float(outs[0].abs().max())
    n, K_, O_ = 300, 736, 2080
    x = synth.normal_tensor((n, K_), 1.0, seed=8, dtype=torch.bfloat16).cuda()
    w = synth.uniform_tensor((O_, K_), float(np.sqrt(3.0 / K_)), seed=9, tensor_id=1, dtype=torch.bfloat16).cuda()
    ref = x.double() @ w.double().T
    wp = tr.pack_weight(w)
    ws = torch.empty((n + 15) // 16 * 16 * K_ * 2 + 512 + 2 * n * O_ * 4 + 528, dtype=torch.uint8, device="cuda")
    for splits in (1, 2):
        for a, b in ((_off_16(wp), ws), (wp, ws[8:])):
            y = torch.full((n, O_), float("nan"), device="cuda")
            ctx.op_linear(x, a, y, b, packed=True, splits=splits)
            assert float((y.double() - ref).abs().max()) < 2e-5 * np.sqrt(K_)
    ctx.close()


def test_linear_row_limits():
    """Packed weights take up to TR_PREFILL_ROWS rows (the prompt-ingestion kernel above TR_MAX_NODES), row-major
    ones TR_MAX_NODES; one more is TR_EINVAL, on the host, before any launch."""
    require_gpu()
    ctx = tr.Context(16, 8, [-1], [-1], 1)
    K_, O_ = 64, 32
    w = synth.uniform_tensor((O_, K_), 0.1, seed=1, tensor_id=0, dtype=torch.bfloat16).cuda()
    wp = tr.pack_weight(w)
    ws = torch.empty(1 << 20, dtype=torch.uint8, device="cuda")
    for n, packed, ok in ((512, True, True), (513, True, False), (128, False, True), (129, False, False)):
        x = torch.zeros(n, K_, dtype=torch.bfloat16, device="cuda")
        y = torch.zeros(n, O_, dtype=torch.float32, device="cuda")
        if ok:
            ctx.op_linear(x, wp if packed else w, y, ws, packed=packed, splits=1)
        else:
            with pytest.raises(tr.TRError) as e:
                ctx.op_linear(x, wp if packed else w, y, ws, packed=packed, splits=1)
            assert e.value.status == tr.TR_EINVAL
    torch.cuda.synchronize()


def test_linear_packed_every_planned_variant():
    """Every (row tiles, weight tiles per workgroup) pair the operation's planner can choose over a grid of shapes,
    with 1, 2 and 4 K-splits, is run once at the cheapest shape that selects it, against a float64 matrix
    product."""
    require_gpu()
    chosen = {}
    for n in (1, 5, 16, 17, 33, 48, 64, 65, 80, 96, 97, 112, 128):
        for K_ in (256, 1024, 2048, 4096, 8192, 11008):
            for O_ in (64, 256, 1024, 2048, 4096, 8192, 12288, 32000):
                if K_ * O_ > 140e6:
                    continue
                for ms in (1, 2, 4):
                    p, _ = tr.plan_linear(n, K_, O_, ms)
                    key, cost = ((n + 15) // 16, p, ms), n * K_ * O_   # the op runs exactly ms K-splits
                    if key not in chosen or cost < chosen[key][0]:
                        chosen[key] = (cost, (n, K_, O_, ms))
    assert len(chosen) >= 70, len(chosen)
    ctx = tr.Context(16, 8, [-1], [-1], 1)
    for key, (_, (n, K_, O_, ms)) in sorted(chosen.items()):
        say("linear variant", key, "shape", n, K_, O_, "max splits", ms)
        x = synth.normal_tensor((n, K_), 1.0, seed=n + K_, dtype=torch.bfloat16)
        w = synth.uniform_tensor((O_, K_), float(np.sqrt(3.0 / K_)), seed=7, tensor_id=O_, dtype=torch.bfloat16)
        y = torch.zeros(n, O_, dtype=torch.float32, device="cuda")
        ws = torch.empty(((n + 15) // 16 * 16 * K_ * 2 + 512 + ms * n * O_ * 4 + 512), dtype=torch.uint8, device="cuda")
        ctx.op_linear(x.cuda(), tr.pack_weight(w.cuda()), y, ws, packed=True, splits=ms)
        ref = x.double().numpy() @ w.double().numpy().T
        err = np.abs(y.cpu().numpy() - ref).max()
        assert err < 2e-5 * np.sqrt(K_), (key, n, K_, O_, ms, err)
    ctx.close()


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_linear_generic_matches_oracle_matmul(dtype):
    require_gpu()
    n, K_, O_ = 45, 344, 130
    x = synth.normal_tensor((n, K_), 1.0, seed=1, dtype=dtype)
    w = synth.uniform_tensor((O_, K_), float(np.sqrt(3.0 / K_)), seed=5, tensor_id=3, dtype=dtype)
    ctx = tr.Context(16, 8, [-1], [-1], 1)
    y = torch.zeros(n, O_, dtype=torch.float32, device="cuda")
    ctx.op_linear(x.cuda(), w.cuda(), y)
    ref = x.double().numpy() @ w.double().numpy().T
    assert np.abs(y.cpu().numpy() - ref).max() < 2e-5 * np.sqrt(K_)


def test_pack_rejects_bad_sizes():
    require_gpu()
    w = torch.zeros(48, 64, dtype=torch.bfloat16, device="cuda")
    with pytest.raises(tr.TRError) as e:
        tr.pack_weight(w)                                      # 48 is not a multiple of 32
    assert e.value.status == tr.TR_EINVAL


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("n,K,O", [(1, 1, 1), (15, 128, 1024), (16, 344, 17), (17, 385, 33), (33, 31, 16), (64, 500, 20),
                                   (65, 1027, 15), (128, 192, 130),
                                   # one, two and four row tiles a workgroup, on both sides of 256 workgroups
                                   (64, 64, 1024), (65, 40, 1024), (48, 96, 2048), (64, 64, 2049), (113, 40, 1024), (128, 33, 1040)])
def test_row_major_linear_edges(dtype, n, K, O):
    """Row-major projections around the kernel's units (16 outputs, 1 / 2 / 4 row tiles per workgroup, k-steps of 64
    bytes dealt to four waves, 16-byte chunks that end inside or straddle a row's end, rows that start off 16 bytes)."""
    require_gpu()
    say("row-major linear", dtype, n, K, O)
    x = synth.normal_tensor((n, K), 1.0, seed=K, dtype=dtype)
    w = synth.normal_tensor((O, K), 1.0, seed=O + 1, dtype=dtype)
    ctx = tr.Context(64, 8, [-1], [-1], 1)
    y = torch.full((n, O), float("nan"), device="cuda")
    ctx.op_linear(x.cuda(), w.cuda(), y)
    want = x.double() @ w.double().t()
    # products are exact in float32 for bf16 and rounded once for float32; K - 1 sums, each off by half an ulp
    bound = (K + 1) * 2.0 ** -24 * (x.double().abs() @ w.double().abs().t())
    assert bool(((y.cpu().double() - want).abs() <= bound).all())
    ctx.close()


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("n,K,O", [(1, 128, 384), (15, 344, 128), (80, 512, 512), (80, 1024, 512), (64, 4096, 512), (128, 4096, 2048),
                                   (33, 2048, 2048), (16, 11008, 512)])
def test_row_major_linear_accumulates_in_short_chains(dtype, n, K, O):
    """Row-major projections against float64, all errors together: no more than 64 running sums of K / 64 products each and
    a tree over them leave, whose roundings of half an ulp add up as a random walk (one running sum per wave leaves up to
    three times as much)."""
    require_gpu()
    say("row-major linear, precision", dtype, n, K, O)
    x = synth.normal_tensor((n, K), 1.0, seed=K, dtype=dtype).cuda()
    w = synth.normal_tensor((O, K), 1.0, seed=O + 1, dtype=dtype).cuda()
    ctx = tr.Context(64, 8, [-1], [-1], 1)
    y = torch.zeros(n, O, device="cuda")
    ctx.op_linear(x, w, y)
    want = x.double() @ w.double().t()
    err = float((y.double() - want).norm() / want.norm())
    say("relative error", err)
    assert err < 2.0 ** -24 * (1.3 + np.sqrt(K) / 32)
    ctx.close()
