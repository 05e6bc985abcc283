"""GPU parity: the HIP library against the fp64 CPU oracle, element by element, through the C ABI.

Bars (written here, from the benchmark spec): routing indices, counts, permutation and unpacked
codes bit-exact; layer outputs within 5e-3 relative Frobenius error.
"""
import numpy as np
import pytest

from oracle import fixtures
from oracle import moe_lrc_oracle as orc
from workload import configs, synth

pytestmark = pytest.mark.gpu

TOL = 5e-3


@pytest.fixture(scope="module")
def amd():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    import paper_2512_17073_amd as amd
    amd.lib()          # raises if the HIP library is not built: no fallback
    return amd


def _to_np(t):
    import torch
    if t.dtype == torch.bfloat16:
        return t.float().cpu().numpy().astype(np.float64)
    return t.cpu().numpy()


def _build(amd, cfg, method="exact", residency=0, **kw):
    layer = fixtures.build_layer(cfg, method=method, **kw)
    L = amd.Layer.from_config(cfg, residency=residency)
    L.load(layer)
    return layer, L


SMALL = {
    "tiny": configs.TINY,
    "tiny_b2": configs.TINY.with_(bits=2, name="tiny_b2"),
    "tiny_b4_n2": configs.TINY.with_(bits=4, top_n=2, rank=16, name="tiny_b4_n2"),
    # > 32 rows per expert: exercises two row tiles and the row-chunk loop, ragged tails
    "tiny_T200": configs.TINY.with_(tokens=200, name="tiny_T200"),
    # several 128-row chunks per expert with a ragged last one; a rank that is no multiple of 16 or 32
    # (padding columns of the factors) at 4 bit
    "tiny_T700_r40": configs.TINY.with_(tokens=700, rank=40, bits=4, name="tiny_T700_r40"),
    # thousands of rows with the rank-r term: 32 rows per block in both (in A) launches
    "tiny_T8300_r64": configs.TINY.with_(tokens=8300, rank=64, name="tiny_T8300_r64"),
    # heavily skewed routing at decode size: some experts get more than 32 rows (several passes of
    # the decode kernel), others none
    "tiny_skew": configs.TINY.with_(tokens=44, gate_kind="unit", gate_std=1.0, zipf_s=3.0, name="tiny_skew"),
    # the largest quantization group (one scale/zero per 256 inputs = one per k-step of a lane row)
    "tiny_g256": configs.TINY.with_(group=256, bits=2, tokens=20, name="tiny_g256"),
    # a single expert: every token routes to it with weight 1, k = n = 1
    "tiny_e1": configs.TINY.with_(n_experts=1, top_k=1, top_n=1, tokens=40, name="tiny_e1"),
    "tiny_T1": configs.TINY.with_(tokens=1, name="tiny_T1"),
    # the limits of the configuration: 256 experts, k = 16 (n = 15), some experts without rows
    "tiny_e256_k16": configs.TINY.with_(n_experts=256, top_k=16, top_n=15, tokens=40, ffn=256, rank=8, name="tiny_e256_k16"),
    "tiny_renorm": configs.TINY.with_(renormalize=1, tokens=33, name="tiny_renorm"),
    # DeepSeek-shaped: shared experts at 4 bit, FFN 1408 (not a multiple of the 256-row k-step), k=6
    "deepseek_small": configs.DEEPSEEK.with_(hidden=512, n_experts=16, tokens=70, name="deepseek_small"),
    # Qwen3-shaped: group 128, many experts, k=8, Zipf-skewed routing
    "qwen3_small": configs.QWEN3.with_(hidden=512, ffn=768, tokens=48, name="qwen3_small"),
}


@pytest.fixture(scope="module", params=list(SMALL))
def case(request, amd):
    cfg = SMALL[request.param]
    print(f"\n[case {cfg.name}] building fixture", flush=True)
    layer, L = _build(amd, cfg)
    x_bits = synth.make_tokens(cfg)
    ref = fixtures.oracle_forward(cfg, layer, x_bits)
    assert (ref["route"]["margin"] > 1e-9).all(), "fixture has a near-tie; routing would be undecidable"
    x = amd.bf16_tensor(x_bits)
    yield cfg, layer, L, x_bits, x, ref
    L.close()


def test_unpacked_codes_bit_exact(case, amd):
    cfg, layer, L, *_ = case
    for e in range(cfg.n_experts + cfg.n_shared):
        for mat in (0, 1, 2):
            got = _to_np(L.debug_unpack(e, mat))
            np.testing.assert_array_equal(got, layer["experts"][e][mat]["codes"], err_msg=f"expert {e} mat {mat}")


def test_route_bit_exact(case):
    cfg, layer, L, x_bits, x, ref = case
    idx, w = L.route(x)
    np.testing.assert_array_equal(_to_np(idx), ref["route"]["idx"])
    np.testing.assert_allclose(_to_np(w), ref["route"]["w"], rtol=2e-6, atol=1e-30)


def test_permute_bit_exact(case):
    cfg, layer, L, x_bits, x, ref = case
    idx, _ = L.route(x)
    counts, offsets, row_pair, pair_row, comp = L.permute(idx)
    p = ref["perm"]
    np.testing.assert_array_equal(_to_np(counts), p["counts"])
    np.testing.assert_array_equal(_to_np(offsets), p["offsets"])
    np.testing.assert_array_equal(_to_np(row_pair), p["row_pair"])
    np.testing.assert_array_equal(_to_np(pair_row), p["pair_row"])
    np.testing.assert_array_equal(_to_np(comp), p["comp_counts"])


@pytest.mark.parametrize("experts,top_k,top_n,tokens", [(8, 2, 1, 4097), (8, 2, 1, 20000), (128, 8, 2, 1025), (128, 8, 3, 7777),
                                                         (61, 6, 2, 3000)])
def test_permute_by_several_blocks(amd, experts, top_k, top_n, tokens):
    """Above 8192 pairs the grouping runs as two launches of several blocks: bit-exact against the
    oracle for ragged sizes, skewed expert loads and experts without rows, twice in a row, then once
    more with a smaller batch (another number of blocks)."""
    import torch
    cfg = configs.TINY.with_(n_experts=experts, top_k=top_k, top_n=top_n, tokens=tokens, rank=0, name="perm_blocks")
    L = amd.Layer.from_config(cfg, max_tokens=tokens)
    rng = np.random.default_rng(experts * 1000 + tokens)
    for T in (tokens, tokens, max(8192 // top_k + 1, tokens // 2)):
        # distinct experts per token, skewed towards a few; expert 1 never chosen
        pw = rng.random(experts) ** 4
        pw[1 % experts] = 0.0
        pw /= pw.sum()
        idx = np.stack([rng.choice(experts, size=top_k, replace=False, p=pw) for _ in range(T)]).astype(np.int32)
        p = orc.permute(idx, experts, top_n)
        got = L.permute(torch.from_numpy(idx).cuda())
        for g, key in zip(got, ("counts", "offsets", "row_pair", "pair_row", "comp_counts")):
            np.testing.assert_array_equal(_to_np(g), p[key], err_msg=f"T={T} {key}")
    L.close()


def test_expert_ffn_and_combine(case):
    cfg, layer, L, x_bits, x, ref = case
    idx, w = L.route(x)
    counts, offsets, row_pair, pair_row, comp = L.permute(idx)
    y = L.expert_ffn(x, offsets, row_pair)
    err_rows = orc.rel_frobenius(_to_np(y), ref["y_rows"])
    out = L.combine(y, w, pair_row, x)
    err_out = orc.rel_frobenius(_to_np(out), ref["out"])
    per_tok = np.linalg.norm(_to_np(out) - ref["out"], axis=1) / np.linalg.norm(ref["out"], axis=1)
    print(f"[{cfg.name}] y_rows rel err {err_rows:.2e}, out rel err {err_out:.2e}, worst token {per_tok.max():.2e}")
    assert err_rows <= TOL and err_out <= TOL
    st = L.stats()
    from oracle import compress
    want = compress.staged_bytes(ref["perm"]["counts"], ref["perm"]["comp_counts"], cfg.hidden, cfg.ffn,
                                 cfg.bits, cfg.group, cfg.rank)
    P = 3 * cfg.hidden * cfg.ffn
    assert st["active_experts"] == want["active_experts"]
    assert st["comp_experts"] == (want["comp_experts"] if cfg.rank and cfg.top_n else 0)
    assert st["bytes_codes"] == want["bytes_codes"] + cfg.n_shared * P * cfg.shared_bits // 8
    assert st["bytes_meta"] == want["bytes_meta"] + cfg.n_shared * (P // cfg.group * 4)
    assert st["bytes_factors"] == (want["bytes_factors"] if cfg.top_n else 0)


def test_forward_matches_four_calls_and_is_deterministic(case):
    import torch
    cfg, layer, L, x_bits, x, ref = case
    idx, w = L.route(x)
    counts, offsets, row_pair, pair_row, comp = L.permute(idx)
    y = L.expert_ffn(x, offsets, row_pair)
    out4 = L.combine(y, w, pair_row, x).clone()
    out_a = L.forward(x).clone()
    out_b = L.forward(x).clone()
    assert torch.equal(out_a.view(torch.int16), out_b.view(torch.int16)), "two runs differ"
    # the composite equals the four calls up to rounding: it may add the fp32 K-block partial sums of
    # W2 in the combine instead of reading expert rows rounded to bf16 (one bf16 rounding, 2^-9, fewer)
    assert orc.rel_frobenius(_to_np(out_a), _to_np(out4)) <= 2.5e-3, "forward differs from the four calls by more than a rounding"
    e_fwd, e_four = orc.rel_frobenius(_to_np(out_a), ref["out"]), orc.rel_frobenius(_to_np(out4), ref["out"])
    print(f"[{cfg.name}] forward {e_fwd:.2e}, four calls {e_four:.2e}")
    assert e_fwd <= TOL and e_fwd <= e_four * 1.05 + 1e-4


def test_workspace_contents_do_not_matter(case):
    """The caller's workspace may hold anything: the forward pass (and the four calls) give the same
    bits after it was filled with 0xFF bytes (NaN patterns as fp16 or fp32, -1 as integers) as after
    zeros.  This covers the rows the kernels stage in place of rows past an expert's last one (kept
    at zero by the preparing launch of the same call) and every table the launches hand each other."""
    import torch
    cfg, layer, L, x_bits, x, ref = case
    T = x.shape[0]
    outs = []
    for fill in (0x00, 0xFF, 0x7E):
        L.workspace(T).fill_(fill)
        out = L.forward(x).clone()
        L.workspace(T).fill_(fill)
        idx, w = L.route(x)
        counts, offsets, row_pair, pair_row, comp = L.permute(idx)
        y = L.expert_ffn(x, offsets, row_pair)
        out4 = L.combine(y, w, pair_row, x).clone()
        outs.append((out, out4))
    for out, out4 in outs[1:]:
        assert torch.equal(out.view(torch.int16), outs[0][0].view(torch.int16)), "forward depends on what the workspace held"
        assert torch.equal(out4.view(torch.int16), outs[0][1].view(torch.int16)), "the four calls depend on what the workspace held"
    assert orc.rel_frobenius(_to_np(outs[1][0]), ref["out"]) <= TOL


def test_constructed_ties(amd):
    # duplicated gate rows and an all-zero token: lower index wins, on the GPU as in the oracle
    cfg = configs.TINY.with_(top_k=3, top_n=1, tokens=40, rank=0, name="ties")
    rng = np.random.default_rng(3)
    wg = rng.normal(size=(cfg.n_experts, cfg.hidden)).astype(np.float32)
    wg[5] = wg[2]; wg[7] = wg[2]
    xf = rng.normal(size=(cfg.tokens, cfg.hidden)).astype(np.float32)
    xf[0] = 0.0
    wg_bits, x_bits = synth.f32_to_bf16_bits(wg), synth.f32_to_bf16_bits(xf)
    ref = orc.route(x_bits, wg_bits, cfg.top_k)
    assert (ref["margin"] == 0).any()
    L = amd.Layer.from_config(cfg)
    L.set_gate(wg_bits)
    idx, w = L.route(amd.bf16_tensor(x_bits))
    np.testing.assert_array_equal(_to_np(idx), ref["idx"])
    np.testing.assert_allclose(_to_np(w), ref["w"], rtol=2e-6)
    assert list(_to_np(idx)[0]) == [0, 1, 2]
    L.close()


def test_n0_equals_rank0_layer_bitwise(amd):
    import torch
    cfg = configs.TINY.with_(top_n=0, name="n0")
    layer, L = _build(amd, cfg)
    cfg0 = configs.TINY.with_(rank=0, name="r0")
    layer0 = {"wg": layer["wg"], "bias": layer["bias"],
              "experts": [{m: dict(ex[m], A=None, B=None) for m in (0, 1, 2)} for ex in layer["experts"]]}
    L0 = amd.Layer.from_config(cfg0)
    L0.load(layer0)
    x_bits = synth.make_tokens(cfg)
    x = amd.bf16_tensor(x_bits)
    a, b = L.forward(x).clone(), L0.forward(x).clone()
    assert torch.equal(a.view(torch.int16), b.view(torch.int16))
    ref = fixtures.oracle_forward(cfg, layer, x_bits)
    assert orc.rel_frobenius(_to_np(a), ref["out"]) <= TOL
    L.close(); L0.close()


def test_large_scale_and_degenerate_groups(amd):
    # scales >= 1 (constant groups get scale 1) must not overflow the fp16 metadata
    cfg = configs.TINY.with_(rank=0, top_n=0, bits=2, name="degenerate")
    layer = fixtures.build_layer(cfg)
    ex = layer["experts"][0]
    for m in (0, 1, 2):
        ex[m]["codes"][:64, :] = 0
        s = ex[m]["scale"].view(np.float16).copy(); z = ex[m]["zero"].view(np.float16).copy()
        s[0, :] = 1.0; z[0, :] = 0.01
        s[1, ::2] = 3.0
        ex[m]["scale"], ex[m]["zero"] = s.view(np.uint16), z.view(np.uint16)
    L = amd.Layer.from_config(cfg)
    L.load(layer)
    x_bits = synth.make_tokens(cfg)
    ref = fixtures.oracle_forward(cfg, layer, x_bits)
    out = L.forward(amd.bf16_tensor(x_bits))
    assert np.isfinite(_to_np(out)).all()
    assert orc.rel_frobenius(_to_np(out), ref["out"]) <= TOL
    L.close()


def test_staged_mode_matches_resident(amd):
    import torch
    cfg = configs.TINY.with_(tokens=5, name="staged")     # few tokens: some experts stay on the host
    layer = fixtures.build_layer(cfg)
    # The device slots of a staged layer start out with whatever the allocation held.  Make that
    # NaN factors (a resident layer with poisoned factors, destroyed right before): an expert whose
    # factors are not brought in must not touch its factor slot.
    import copy
    poison = copy.deepcopy(layer)
    for ex in poison["experts"]:
        for a in ex.values():
            if a.get("A") is not None and np.size(a["A"]):
                a["A"] = np.full_like(a["A"], 0x7FC0)
                a["B"] = np.full_like(a["B"], 0x7FC0)
    Lp = amd.Layer.from_config(cfg, max_tokens=16)
    Lp.load(poison)
    Lp.close()
    Ls = amd.Layer.from_config(cfg, max_tokens=16, residency=amd.STAGED)
    Lr = amd.Layer.from_config(cfg, max_tokens=16)
    Lr.load(layer); Ls.load(layer)
    x_bits = synth.make_tokens(cfg)
    x = amd.bf16_tensor(x_bits)
    a, b = Lr.forward(x).clone(), Ls.forward(x).clone()
    assert torch.equal(a.view(torch.int16), b.view(torch.int16))
    ref = fixtures.oracle_forward(cfg, layer, x_bits)
    from oracle import compress
    want = compress.staged_bytes(ref["perm"]["counts"], ref["perm"]["comp_counts"], cfg.hidden, cfg.ffn,
                                 cfg.bits, cfg.group, cfg.rank)
    st = Ls.stats()
    assert want["active_experts"] < cfg.n_experts
    for k in ("active_experts", "comp_experts", "bytes_codes", "bytes_meta", "bytes_factors"):
        assert st[k] == want[k], k
    assert st["stage_ms"] > 0
    # a second batch that routes elsewhere must bring in its own experts
    cfg2 = cfg.with_(seed=99, tokens=7)
    x2_bits = synth.make_tokens(cfg2)
    x2 = amd.bf16_tensor(x2_bits)
    assert torch.equal(Lr.forward(x2).view(torch.int16), Ls.forward(x2).view(torch.int16))
    np.testing.assert_array_equal(_to_np(Ls.debug_unpack(3, 1)), layer["experts"][3][1]["codes"])
    Lr.close(); Ls.close()


def test_long_k_several_staging_phases(amd):
    """An FFN width of 36864: the decode flavour's W2 launch splits its K into 8 K-blocks of 18
    k-steps, i.e. two staging phases per block with one row tile and three with two (the Mixtral
    shape has one and two).  Two experts, k = 2: each holds every token, so 20 tokens take the
    two-row-tile body and their first 10 the one-row-tile body."""
    # the same for the fused projection, whose K is the hidden size and is not split into K-blocks:
    # the largest hidden size a layer accepts gives four and eight phases
    # (and 150 tokens: the grouped-GEMM flavour, two chunks per expert, over the same long K)
    for cfg in (configs.TINY.with_(n_experts=2, top_k=2, top_n=1, tokens=150, ffn=36864, bits=2, rank=8, name="long_k"),
                configs.TINY.with_(n_experts=2, top_k=2, top_n=1, tokens=150, hidden=16384, ffn=256, bits=3, rank=8, name="long_h")):
        layer, L = _build(amd, cfg)
        x_bits = synth.make_tokens(cfg)
        for T in (20, 10, 150):
            ref = fixtures.oracle_forward(cfg.with_(tokens=T), layer, x_bits[:T])
            out = L.forward(amd.bf16_tensor(x_bits[:T]))
            err = orc.rel_frobenius(_to_np(out), ref["out"])
            print(f"[{cfg.name}] T={T}: {err:.2e}")
            assert err <= TOL
        L.close()


def test_empty_batch(amd):
    """T = 0: every hot-path call returns without touching its per-token buffers (empty tensors have
    null data pointers); the grouping still reports zero rows for every expert."""
    import torch
    cfg = configs.TINY
    layer, L = _build(amd, cfg)
    x0 = torch.empty((0, cfg.hidden), dtype=torch.bfloat16, device="cuda")
    idx, w = L.route(x0)
    assert idx.shape == (0, cfg.top_k) and w.shape == (0, cfg.top_k)
    counts, offsets, row_pair, pair_row, comp = L.permute(idx)
    torch.cuda.synchronize()
    assert not counts.any() and not offsets.any() and not comp.any()
    y = L.expert_ffn(x0, offsets, row_pair)
    out = L.combine(y, w, pair_row, x0)
    assert y.shape == (0, cfg.hidden) and out.shape == (0, cfg.hidden)
    assert L.forward(x0).shape == (0, cfg.hidden)
    sentinel = torch.full((4, cfg.hidden), 1.5, dtype=torch.bfloat16, device="cuda")
    L.forward(x0, out=sentinel[:0])
    torch.cuda.synchronize()
    assert (sentinel == 1.5).all()
    # and the layer still works afterwards
    x_bits = synth.make_tokens(cfg)
    ref = fixtures.oracle_forward(cfg, layer, x_bits)
    assert orc.rel_frobenius(_to_np(L.forward(amd.bf16_tensor(x_bits))), ref["out"]) <= TOL
    L.close()


def test_hot_path_argument_errors(amd):
    import torch
    cfg = configs.TINY
    L = amd.Layer.from_config(cfg)
    x = amd.bf16_tensor(synth.make_tokens(cfg))
    with pytest.raises(amd.MoeLrcError) as ei:
        L.route(x)                                # gate not uploaded
    assert ei.value.code == -3
    wg, _ = synth.make_gate(cfg)
    L.set_gate(wg)
    with pytest.raises(amd.MoeLrcError) as ei:
        L.forward(x)                              # experts not uploaded
    assert ei.value.code == -3
    big = torch.zeros((cfg.tokens + 1, cfg.hidden), dtype=torch.bfloat16, device="cuda")
    with pytest.raises(amd.MoeLrcError) as ei:
        L.route(big)                              # T > max_tokens
    assert ei.value.code == -3
    with pytest.raises(amd.MoeLrcError) as ei:
        L.set_expert(0, 0, np.full((256, 512), 9, np.uint8), np.zeros((4, 512), np.uint16),
                     np.zeros((4, 512), np.uint16), np.zeros((256, 8), np.uint16), np.zeros((8, 512), np.uint16))
    assert ei.value.code == -1                    # code out of range for 3 bits
    L.close()


@pytest.mark.parametrize("name", ["tiny", "deepseek_small"])
def test_forward_under_graph_capture_replays_like_eager(amd, name):
    """moe_lrc_forward allocates nothing, never synchronises in resident mode and clears nothing with
    a memset, so it can be captured into a HIP graph (with shared experts the capture forks to the
    layer's side stream and joins again).  Every replay, with the program's own eager work and
    synchronisations in between, must give the bits of the eager call on the same tokens."""
    import torch
    cfg = SMALL[name]
    layer = fixtures.build_layer(cfg)
    L = amd.Layer.from_config(cfg)
    L.load(layer)
    T = cfg.tokens
    xs = [amd.bf16_tensor(synth.make_tokens(cfg.with_(seed=cfg.seed + 17 * i))) for i in range(3)]
    eager = [L.forward(x).clone() for x in xs]           # (also the warm-up: function attributes are set)
    torch.cuda.synchronize()
    x_static = xs[0].clone()
    out = torch.empty((T, cfg.hidden), dtype=torch.bfloat16, device="cuda")
    ws = L.workspace(T)
    g = torch.cuda.CUDAGraph()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        with torch.cuda.graph(g, stream=side):
            L.forward_raw(x_static.data_ptr(), T, out.data_ptr(), ws.data_ptr(), ws.numel(),
                          torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    for rep in range(2):
        for i, x in enumerate(xs):
            x_static.copy_(x)
            g.replay()
            torch.cuda.synchronize()
            assert torch.equal(out.view(torch.int16), eager[i].view(torch.int16)), (rep, i)
            again = L.forward(x)                          # eager work between the replays
            torch.cuda.synchronize()
            assert torch.equal(again.view(torch.int16), eager[i].view(torch.int16))
    L.close()


def test_route_tiled_path_many_tokens_and_experts(amd):
    """With >= 1024 tokens and >= 128 experts the logits come from the tiled fp64-matrix-core kernel
    (ragged token and expert tiles here: T = 1100, E = 136): indices bit-exact, ties included."""
    cfg = configs.QWEN3.with_(hidden=320, ffn=256, group=64, n_experts=136, tokens=1100, rank=0, top_n=0, name="route_tiled")
    wg, bias = synth.make_gate(cfg)
    wg = wg.copy()
    wg[5] = wg[77]                      # a duplicated gate row: equal logits, the lower index wins
    if bias is not None:
        bias = bias.copy(); bias[5] = bias[77]
    x_bits = synth.make_tokens(cfg)
    ref = orc.route(x_bits, wg, cfg.top_k, cfg.renormalize, bias)
    L = amd.Layer.from_config(cfg)
    L.set_gate(wg, bias)
    idx, w = L.route(amd.bf16_tensor(x_bits))
    np.testing.assert_array_equal(_to_np(idx), ref["idx"])
    np.testing.assert_allclose(_to_np(w), ref["w"], rtol=2e-6, atol=1e-30)
    L.close()


@pytest.mark.parametrize("hidden,experts", [(64, 8), (1024, 64), (2048, 8), (8192, 8), (8192, 64), (16384, 8), (16384, 130)])
def test_route_over_hidden_sizes(amd, hidden, experts):
    """Every variant of the per-token routing kernel (1 to 32 chunks of a row per lane, 4 or 16
    wavefronts per token), up to the largest hidden size a layer accepts: indices bit-exact."""
    cfg = configs.TINY.with_(hidden=hidden, ffn=64, group=64, n_experts=experts, top_k=min(6, experts), top_n=0, rank=0,
                             tokens=9, name=f"route_h{hidden}_e{experts}")
    wg, bias = synth.make_gate(cfg)
    wg = wg.copy()
    wg[1] = wg[experts - 1]             # equal logits: the lower index wins
    x_bits = synth.make_tokens(cfg)
    ref = orc.route(x_bits, wg, cfg.top_k, cfg.renormalize, bias)
    L = amd.Layer.from_config(cfg)
    L.set_gate(wg, bias)
    idx, w = L.route(amd.bf16_tensor(x_bits))
    np.testing.assert_array_equal(_to_np(idx), ref["idx"])
    np.testing.assert_allclose(_to_np(w), ref["w"], rtol=2e-6, atol=1e-30)
    L.close()


def test_route_with_several_blocks_per_token(amd):
    """With few tokens and 128 experts or more, several blocks share a token's gate rows and leave
    their logits in memory for the Top-k launch that follows.  Batches of different sizes, hence
    different numbers of blocks per token, one after the other on one layer: indices bit-exact every
    time, a duplicated gate row and a ragged expert count (136) included."""
    for E in (128, 136):
        cfg = configs.QWEN3.with_(hidden=512, ffn=256, group=64, n_experts=E, tokens=100, rank=0, top_n=0, name=f"route_split_{E}")
        wg, bias = synth.make_gate(cfg)
        wg = wg.copy()
        wg[3] = wg[E - 2]                   # equal logits in different blocks' shares: the lower index wins
        if bias is not None:
            bias = bias.copy(); bias[3] = bias[E - 2]
        x_bits = synth.make_tokens(cfg)
        ref = orc.route(x_bits, wg, cfg.top_k, cfg.renormalize, bias)
        L = amd.Layer.from_config(cfg)
        L.set_gate(wg, bias)
        x = amd.bf16_tensor(x_bits)
        for T in (1, 100, 3, 16, 1, 64, 17, 100):
            idx, w = L.route(x[:T])
            np.testing.assert_array_equal(_to_np(idx), ref["idx"][:T], err_msg=f"E={E} T={T}")
            np.testing.assert_allclose(_to_np(w), ref["w"][:T], rtol=2e-6, atol=1e-30)
        L.close()


@pytest.mark.parametrize("tokens,experts,hidden", [(1001, 60, 1216), (2047, 17, 2112)])
def test_route_tiled_with_ragged_sizes(amd, tokens, experts, hidden):
    """Batches that are routed in tiles of 16 tokens x 16 experts (at least 128 tiles and 2^26 products) at sizes that fill
    neither: a last tile of tokens and of experts, shares of the hidden size that end inside a batch of
    chunks (hidden / 8 no multiple of 128), a duplicated gate row.  Indices bit-exact; and a forward on tokens
    of very different magnitudes, which takes the exponents this kernel writes on its way."""
    import torch
    cfg = configs.TINY.with_(hidden=hidden, ffn=128, n_experts=experts, top_k=3, top_n=1, rank=16, tokens=tokens, gate_kind="unit", gate_std=1.5,
                             name=f"route_tiled_{tokens}_{experts}_{hidden}")
    assert (tokens + 15) // 16 * ((experts + 15) // 16) >= 128 and tokens * experts * hidden >= 1 << 26
    layer = fixtures.sample_layer(cfg)
    layer["wg"] = layer["wg"].copy()
    layer["wg"][3] = layer["wg"][experts - 2]       # equal logits in different tiles: the lower index wins
    x_bits = synth.make_tokens(cfg)
    scale = np.array([(-1) ** t * (3 * t % 37) for t in range(tokens)], dtype=np.int64)
    zero = (x_bits & 0x7fff) == 0
    x_bits = np.where(zero, x_bits, x_bits.astype(np.int64) + (scale[:, None] << 7)).astype(np.uint16)      # times 2^scale
    x_bits[tokens - 2] = 0                          # a token of zeros: all logits equal
    ref = fixtures.oracle_forward(cfg, layer, x_bits)
    L = amd.Layer.from_config(cfg)
    L.load(layer)
    x = amd.bf16_tensor(x_bits)
    idx, w = L.route(x)
    np.testing.assert_array_equal(_to_np(idx), ref["route"]["idx"])
    np.testing.assert_allclose(_to_np(w), ref["route"]["w"], rtol=2e-6, atol=1e-30)
    out = _to_np(L.forward(x))
    torch.cuda.synchronize()
    norm = np.linalg.norm(ref["out"], axis=1)
    err = np.linalg.norm(out - ref["out"], axis=1)[norm > 0] / norm[norm > 0]
    print(f"\n[{cfg.name}] worst token {err.max():.2e}", flush=True)
    assert err.max() <= 4 * TOL and np.abs(out[norm == 0]).max(initial=0.0) == 0.0      # (per token: the worst of thousands)
    L.close()


@pytest.mark.parametrize("tokens", [16, 300])
def test_rank_per_projection_from_kurtosis(amd, tokens):
    """Section 3.1 step 1: the rank budget is spread over the expert matrices by their kurtosis, so
    every projection has a rank of its own (0 included, W1 and W3 of one expert may differ).
    Decode flavour (16 tokens) and grouped-GEMM flavour (300 tokens), resident and staged; the
    staged mode moves only the ranks uploaded."""
    import torch
    cfg = configs.TINY.with_(rank=32, tokens=tokens, name=f"ranks_T{tokens}")
    ranks = fixtures.kurtosis_ranks(cfg, 10, (0, 8, 16, 32))
    assert len(set(ranks.ravel().tolist())) >= 3 and (ranks[:, 0] != ranks[:, 1]).any()
    layer = fixtures.build_layer(cfg, ranks=ranks)
    x_bits = synth.make_tokens(cfg)
    x = amd.bf16_tensor(x_bits)
    ref = fixtures.oracle_forward(cfg, layer, x_bits)
    Lr = amd.Layer.from_config(cfg)
    Ls = amd.Layer.from_config(cfg, residency=amd.STAGED)
    Lr.load(layer); Ls.load(layer)
    out_r = Lr.forward(x).clone()
    torch.cuda.synchronize()
    out_s = Ls.forward(x).clone()
    torch.cuda.synchronize()
    err = orc.rel_frobenius(_to_np(out_r), ref["out"])
    print(f"\n[ranks_T{tokens}] ranks {ranks.tolist()} out rel err {err:.2e}", flush=True)
    assert err <= TOL
    assert torch.equal(out_r.view(torch.int16), out_s.view(torch.int16))
    st = Ls.stats()
    comp = np.asarray(ref["perm"]["comp_counts"]) > 0
    assert st["bytes_factors"] == int((ranks[comp].sum(axis=1) * (cfg.hidden + cfg.ffn) * 2).sum())
    # re-uploading a projection with a smaller rank leaves no trace of the larger one
    e = int(np.argmax(ranks[:, 0] == 32))
    a = dict(layer["experts"][e][0])
    Lr.set_expert(e, 0, a["codes"], a["scale"], a["zero"], None, None, rank=0)
    layer2 = {"wg": layer["wg"], "bias": layer["bias"], "experts": [dict(ex) for ex in layer["experts"]]}
    layer2["experts"][e][0] = dict(a, A=None, B=None, rank=0)
    ref2 = fixtures.oracle_forward(cfg, layer2, x_bits)
    assert orc.rel_frobenius(_to_np(Lr.forward(x)), ref2["out"]) <= TOL
    Lr.close(); Ls.close()


@pytest.mark.parametrize("tokens,rank", [(16, 16), (300, 32), (40, 24), (24, 72), (700, 64)])
def test_int3_factors(amd, tokens, rank):
    """Section 3.1 step 2 stores the factor pairs at INT3: uploaded as 3-bit codes + fp16 scale/zero
    per group of 64, kept at 3 bits in the pinned pool and on the device, and dequantized inside the
    kernels that consume them (both flavours of the (in A) and of the FFN kernels are reached: 16 to
    700 tokens).  Resident and staged layers agree bit for bit and match the oracle on the quantized
    factors; the staged byte counter counts a 4-bit cell + scale/zero per value."""
    import torch
    cfg = configs.TINY.with_(rank=rank, tokens=tokens, bits=2, name=f"int3_T{tokens}_r{rank}")
    layer = fixtures.build_layer(cfg, int3_factors=True)
    x_bits = synth.make_tokens(cfg)
    x = amd.bf16_tensor(x_bits)
    ref = fixtures.oracle_forward(cfg, layer, x_bits)
    Lr = amd.Layer.from_config(cfg)
    Ls = amd.Layer.from_config(cfg, residency=amd.STAGED)
    Lr.load(layer); Ls.load(layer)
    out_r = Lr.forward(x).clone()
    torch.cuda.synchronize()
    out_s = Ls.forward(x).clone()
    torch.cuda.synchronize()
    err = orc.rel_frobenius(_to_np(out_r), ref["out"])
    print(f"\n[{cfg.name}] out rel err {err:.2e}", flush=True)
    assert err <= TOL
    assert torch.equal(out_r.view(torch.int16), out_s.view(torch.int16))
    n_comp = int((np.asarray(ref["perm"]["comp_counts"]) > 0).sum())
    vals = 3 * rank * (cfg.hidden + cfg.ffn)
    assert Ls.stats()["bytes_factors"] == n_comp * (vals * 4 // 8 + vals // 64 * 4)
    # the compensation is really there: without it the output differs by far more than the tolerance
    assert orc.rel_frobenius(_to_np(out_r), fixtures.oracle_forward(cfg.with_(top_n=0), layer, x_bits)["out"]) > 5 * TOL
    Lr.close(); Ls.close()


@pytest.mark.parametrize("tokens", [16, 300, 700])
def test_int3_factors_with_a_rank_per_projection(amd, tokens):
    """Factor pairs at 3 bits whose ranks differ from matrix to matrix (Section 3.1 steps 1 and 2
    together): W1 and W3 of an expert run different numbers of rank steps, some projections have no
    pair at all, and the factor tiles past a projection's own rank add nothing.  All three
    flavour mixes (16, 300, 700 tokens), resident against staged bit for bit."""
    import torch
    cfg = configs.TINY.with_(rank=64, tokens=tokens, bits=2, name=f"int3_ranks_T{tokens}")
    ranks = fixtures.kurtosis_ranks(cfg, 26, (0, 16, 32, 64))
    assert len(set(ranks.ravel().tolist())) >= 3 and (ranks[:, 0] != ranks[:, 1]).any()
    layer = fixtures.build_layer(cfg, ranks=ranks, int3_factors=True)
    x_bits = synth.make_tokens(cfg)
    x = amd.bf16_tensor(x_bits)
    ref = fixtures.oracle_forward(cfg, layer, x_bits)
    Lr = amd.Layer.from_config(cfg)
    Ls = amd.Layer.from_config(cfg, residency=amd.STAGED)
    Lr.load(layer); Ls.load(layer)
    out_r = Lr.forward(x).clone()
    torch.cuda.synchronize()
    out_s = Ls.forward(x).clone()
    torch.cuda.synchronize()
    err = orc.rel_frobenius(_to_np(out_r), ref["out"])
    print(f"\n[{cfg.name}] ranks {ranks.tolist()} out rel err {err:.2e}", flush=True)
    assert err <= TOL
    assert torch.equal(out_r.view(torch.int16), out_s.view(torch.int16))
    assert orc.rel_frobenius(_to_np(out_r), fixtures.oracle_forward(cfg.with_(top_n=0), layer, x_bits)["out"]) > 3 * TOL
    Lr.close(); Ls.close()


def test_mixed_fp16_and_int3_projections_staged(amd):
    """One expert may hold one projection's factors as an fp16 pair and the others at 3 bits: each
    pair lives in its own projection's factor sections, so neither upload disturbs the other, and
    the kernels take the format per projection from the expert table.  Staged and resident layers
    agree bit for bit and match the oracle."""
    import torch
    cfg = configs.TINY.with_(rank=32, tokens=24, bits=2, name="mixed_q3")
    bf = fixtures.build_layer(cfg)
    q3 = fixtures.build_layer(cfg, int3_factors=True)
    experts = []
    for e in range(cfg.n_experts):                       # W1 as a bf16 pair, W3 and W2 at 3 bits (and rotated per expert)
        keep = e % 3
        experts.append({m: (bf if m == keep else q3)["experts"][e][m] for m in (0, 1, 2)})
    layer = {"wg": bf["wg"], "bias": bf["bias"], "experts": experts}
    x_bits = synth.make_tokens(cfg)
    x = amd.bf16_tensor(x_bits)
    ref = fixtures.oracle_forward(cfg, layer, x_bits)
    Lr = amd.Layer.from_config(cfg)
    Ls = amd.Layer.from_config(cfg, residency=amd.STAGED)
    # upload order matters for an overlap bug: 3-bit blobs first on one layer, last on the other
    Lr.load(layer)
    Ls.set_gate(layer["wg"], layer["bias"])
    for e, ex in enumerate(experts):
        for m in (2, 1, 0):
            a = ex[m]
            if a.get("Aq") is not None:
                Ls.set_expert(e, m, a["codes"], a["scale"], a["zero"], None, None, 0)
                Ls.set_expert_factors_quantized(e, m, a["Aq"]["codes"].shape[1], a["Aq"], a["Bq"])
        for m in (0, 1, 2):
            a = ex[m]
            if a.get("Aq") is None:
                Ls.set_expert(e, m, a["codes"], a["scale"], a["zero"], a["A"], a["B"], cfg.rank)
    out_r = Lr.forward(x).clone()
    out_s = Ls.forward(x).clone()
    torch.cuda.synchronize()
    err = orc.rel_frobenius(_to_np(out_r), ref["out"])
    print(f"\n[{cfg.name}] out rel err {err:.2e}", flush=True)
    assert err <= TOL
    assert torch.equal(out_r.view(torch.int16), out_s.view(torch.int16))
    Lr.close(); Ls.close()


def test_stats_path_reports_the_flavour(amd):
    """moe_lrc_stats.path: bit 0 = W1|W3 ran as the grouped GEMM, bit 1 = W2 did."""
    import torch
    cfg = configs.TINY.with_(tokens=700, rank=8, name="path")
    layer = fixtures.sample_layer(cfg)
    L = amd.Layer.from_config(cfg)
    L.load(layer)
    for T, want in ((8, 0), (700, 3)):
        x = amd.bf16_tensor(synth.make_tokens(cfg, T))
        L.forward(x)
        torch.cuda.synchronize()
        assert L.stats()["path"] == want, (T, L.stats()["path"])
    L.close()


@pytest.mark.parametrize("tokens", [16, 100, 300, 700])
def test_ranks_from_the_papers_bucket_up_to_1024(amd, tokens):
    """Section 3.1 step 1 allocates every expert matrix a rank from the bucket {0, 16, 32, 128, 256,
    512, 1024}.  A layer whose projections cycle through the whole bucket (W1, W3 and W2 of one expert
    all different), at 16 tokens (skinny kernels, one row tile), 100 (two row tiles, several passes,
    the (in A) fragments of the large ranks taking the place of the staged activations), 300 (fused
    projection as grouped GEMM, W2 skinny) and 700 (both grouped GEMM, rank steps in chunks), against
    the oracle on the same stored factors; resident and staged layers agree bit for bit."""
    import torch
    bucket = (0, 16, 32, 128, 256, 512, 1024)
    cfg = configs.TINY.with_(rank=1024, tokens=tokens, bits=2, name=f"bucket_T{tokens}")
    layer = fixtures.sample_layer(cfg)
    for e, ex in enumerate(layer["experts"]):
        for m in (0, 1, 2):
            r = bucket[(3 * e + 2 * m) % len(bucket)]
            a = ex[m]
            a["rank"] = r
            a["A"] = np.ascontiguousarray(a["A"][:, :r]) if r else None
            a["B"] = np.ascontiguousarray(a["B"][:r]) if r else None
    x_bits = synth.make_tokens(cfg)
    x = amd.bf16_tensor(x_bits)
    ref = fixtures.oracle_forward(cfg, layer, x_bits)
    Lr = amd.Layer.from_config(cfg)
    Ls = amd.Layer.from_config(cfg, residency=amd.STAGED)
    Lr.load(layer); Ls.load(layer)
    out_r = Lr.forward(x).clone()
    torch.cuda.synchronize()
    out_s = Ls.forward(x).clone()
    torch.cuda.synchronize()
    err = orc.rel_frobenius(_to_np(out_r), ref["out"])
    none = orc.rel_frobenius(_to_np(out_r), fixtures.oracle_forward(cfg.with_(top_n=0), layer, x_bits)["out"])
    print(f"\n[{cfg.name}] out rel err {err:.2e} (the rank terms move the output by {none:.2e})", flush=True)
    assert err <= TOL and none > 10 * TOL
    assert torch.equal(out_r.view(torch.int16), out_s.view(torch.int16))
    Lr.close(); Ls.close()


@pytest.mark.parametrize("hidden,ffn,rank,tokens,kind", [
    (1536, 1600, 120, 300, "same"),        # at most two factor tiles per wavefront; a rank that is no multiple of 16
    (704, 832, 1024, 300, "same"),         # four, several groups of 32; K no multiple of a k-step
    (704, 832, 1024, 300, "bucket"),       # ranks far apart, W1 and W3 of an expert differ, some pairs missing
    (832, 704, 520, 1000, "same"),         # an odd number of factor tiles, several 128-row chunks per expert
    (704, 832, 256, 2400, "int3"),         # pairs at 3 bits, enough rows
])
def test_in_a_with_staged_rows(amd, hidden, ffn, rank, tokens, kind):
    """(x A) and (h A2) of many factor tiles take the two launches that stage the rows (tiles times K past
    20480; 3-bit pairs past 8192 and 4e7 with the rows): the sizes at which its splits change, against
    the oracle, and staged residency bit for bit."""
    import torch
    bucket = (1024, 16, 0, 256, 1024, 32, 512)
    cfg = configs.TINY.with_(hidden=hidden, ffn=ffn, n_experts=4, rank=rank, tokens=tokens, bits=2, name=f"staged_rows_{kind}_{hidden}_r{rank}")
    layer = fixtures.sample_layer(cfg)
    for e, ex in enumerate(layer["experts"]):
        for m in (0, 1, 2):
            a = ex[m]
            if kind == "int3":
                a["Aq"], a["Bq"] = synth.sample_factor_codes(cfg, e, m)
                a["A"] = a["B"] = None
            elif kind == "bucket":
                a["rank"] = r = bucket[(3 * e + 2 * m) % len(bucket)]
                a["A"] = np.ascontiguousarray(a["A"][:, :r]) if r else None
                a["B"] = np.ascontiguousarray(a["B"][:r]) if r else None
    x_bits = synth.make_tokens(cfg)
    x = amd.bf16_tensor(x_bits)
    ref = fixtures.oracle_forward(cfg, layer, x_bits)
    Lr = amd.Layer.from_config(cfg)
    Ls = amd.Layer.from_config(cfg, residency=amd.STAGED)
    Lr.load(layer); Ls.load(layer)
    out_r = Lr.forward(x).clone()
    torch.cuda.synchronize()
    assert Lr.stats()["path"] == 3
    out_s = Ls.forward(x).clone()
    torch.cuda.synchronize()
    err = orc.rel_frobenius(_to_np(out_r), ref["out"])
    none = orc.rel_frobenius(_to_np(out_r), fixtures.oracle_forward(cfg.with_(top_n=0), layer, x_bits)["out"])
    print(f"\n[{cfg.name}] out rel err {err:.2e} (the rank terms move the output by {none:.2e})", flush=True)
    assert err <= TOL and none > 5 * TOL
    assert torch.equal(out_r.view(torch.int16), out_s.view(torch.int16))
    Lr.close(); Ls.close()


@pytest.mark.parametrize("hidden,ffn,rank,tokens,experts,kind", [
    (256, 64, 64, 3, 1, "same"),           # four n-tiles for all blocks: most of them own none
    (256, 64, 8, 1, 2, "int3"),            # one 16-column tile, one row
    (512, 1088, 40, 70, 4, "same"),        # several passes, an odd number of factor tiles
    (320, 4160, 56, 37, 2, "int3"),        # W2 in two K-blocks, 260 n-tiles
    (320, 4160, 64, 21, 2, "bucket"),      # ranks that differ, pairs of W2 missing
    # ranks up to 32 and few enough parts: made by the fused launch (the ones above 32 and (512, 1088) by a launch in between)
    (256, 64, 32, 3, 1, "same"),           # four n-tiles for all blocks: most of them own none
    (512, 128, 24, 70, 4, "same"),         # several passes, eight parts
    (320, 4160, 32, 16, 2, "bucket"),      # W2 in two K-blocks, ranks that differ, pairs of W2 missing
    (320, 8256, 32, 30, 4, "int3"),        # three K-blocks, 128 parts of up to 30 rows
])
def test_h_a2_from_the_fused_launch(amd, hidden, ffn, rank, tokens, experts, kind):
    """(h A2) of decode batches with ranks up to 32 is made by the blocks of the fused projection and added up by
    those of W2, where the parts are few: block shares, K-blocks, passes and ranks at which its indices change, against the oracle."""
    import torch
    bucket = tuple(min(r, rank) for r in (64, 0, 16, 40, 0, 8, 64))
    cfg = configs.TINY.with_(hidden=hidden, ffn=ffn, n_experts=experts, top_k=min(2, experts), rank=rank, tokens=tokens, bits=2,
                             name=f"h_a2_{kind}_{ffn}_r{rank}")
    layer = fixtures.sample_layer(cfg)
    for e, ex in enumerate(layer["experts"]):
        for m in (0, 1, 2):
            a = ex[m]
            if kind == "int3":
                a["Aq"], a["Bq"] = synth.sample_factor_codes(cfg, e, m)
                a["A"] = a["B"] = None
            elif kind == "bucket":
                a["rank"] = r = bucket[(3 * e + 2 * m) % len(bucket)]
                a["A"] = np.ascontiguousarray(a["A"][:, :r]) if r else None
                a["B"] = np.ascontiguousarray(a["B"][:r]) if r else None
    x_bits = synth.make_tokens(cfg)
    x = amd.bf16_tensor(x_bits)
    ref = fixtures.oracle_forward(cfg, layer, x_bits)
    Lr = amd.Layer.from_config(cfg)
    Ls = amd.Layer.from_config(cfg, residency=amd.STAGED)
    Lr.load(layer); Ls.load(layer)
    out_r = Lr.forward(x).clone()
    torch.cuda.synchronize()
    assert Lr.stats()["path"] == 0
    out_s = Ls.forward(x).clone()
    torch.cuda.synchronize()
    err = orc.rel_frobenius(_to_np(out_r), ref["out"])
    none = orc.rel_frobenius(_to_np(out_r), fixtures.oracle_forward(cfg.with_(top_n=0), layer, x_bits)["out"])
    print(f"\n[{cfg.name}] out rel err {err:.2e} (the rank terms move the output by {none:.2e})", flush=True)
    assert err <= TOL and none > 3 * TOL
    assert torch.equal(out_r.view(torch.int16), out_s.view(torch.int16))
    Lr.close(); Ls.close()


@pytest.mark.parametrize("hidden,ffn", [(256, 2176), (2176, 256)])      # 17 n-tiles a block of W1|W3, or of W2: no wavefront shares a unit
@pytest.mark.parametrize("rank,kind,bits", [(40, "same", 4), (72, "int3", 3), (104, "int3", 2), (104, "int3", 4), (136, "same", 2), (200, "bucket", 3)])
def test_rank_steps_of_unshared_units(amd, hidden, ffn, rank, kind, bits):
    """Two to seven rank steps that all are one wavefront's (odd and even numbers, ranks that differ or are 0), of one unit and of two,
    with one row tile and with two, against the oracle."""
    cfg = configs.TINY.with_(hidden=hidden, ffn=ffn, n_experts=32, top_k=4, top_n=2, rank=rank, tokens=160, bits=bits, name=f"unshared_{hidden}_r{rank}_b{bits}")
    layer = fixtures.sample_layer(cfg)
    bucket = (200, 8, 0, 104, 200, 32, 64)
    for e, ex in enumerate(layer["experts"]):
        for m in (0, 1, 2):
            a = ex[m]
            if kind == "int3":
                a["Aq"], a["Bq"] = synth.sample_factor_codes(cfg, e, m)
                a["A"] = a["B"] = None
            elif kind == "bucket":
                a["rank"] = r = bucket[(3 * e + 2 * m) % len(bucket)]
                a["A"] = np.ascontiguousarray(a["A"][:, :r]) if r else None
                a["B"] = np.ascontiguousarray(a["B"][:r]) if r else None
    x_bits = synth.make_tokens(cfg)
    ref = fixtures.oracle_forward(cfg, layer, x_bits)
    rows = np.diff(ref["perm"]["offsets"])
    assert (rows > 16).any() and ((rows > 0) & (rows <= 16)).any()
    L = amd.Layer.from_config(cfg)
    L.load(layer)
    out = _to_np(L.forward(amd.bf16_tensor(x_bits)))
    assert L.stats()["path"] == 0
    none = orc.rel_frobenius(out, fixtures.oracle_forward(cfg.with_(top_n=0), layer, x_bits)["out"])
    assert orc.rel_frobenius(out, ref["out"]) <= TOL and none > 3 * TOL
    L.close()


@pytest.mark.parametrize("experts,top_k,busy,tokens,rank,kind", [
    (8, 2, 2, 160, 256, "same"),           # passes beyond the first: 8, of 32 tiles each, dealt to 128 blocks twice
    (20, 2, 2, 33, 8, "same"),             # one row beyond the first pass of either expert
    (130, 3, 3, 100, 24, "int3"),          # experts of the third group of 64 have them all; an odd number of tiles
    (16, 1, 1, 65, 40, "bucket"),          # one expert has every row; ranks that differ, pairs missing
    (12, 1, 12, 32, 16, "same"),           # no expert can have more than one pass
])
def test_x_a13_of_experts_with_several_passes(amd, experts, top_k, busy, tokens, rank, kind):
    """(x A1 | x A3) of the routed rows where the last `busy` experts take every token: the passes of 32 rows beyond an expert's first
    one, which blocks of their own share, against the oracle and, bit for bit, staged residency, where one block makes them all."""
    import torch
    cfg = configs.TINY.with_(hidden=320, ffn=256, n_experts=experts, top_k=top_k, top_n=top_k, tokens=tokens, bits=2, rank=rank, name=f"busy_{experts}_{tokens}_r{rank}")
    layer = fixtures.sample_layer(cfg)
    layer["bias"] = np.where(np.arange(experts) >= experts - busy, 100.0, 0.0).astype(np.float32)
    bucket = (rank, 0, 16, rank, 8)
    for e, ex in enumerate(layer["experts"]):
        for m in (0, 1, 2):
            a = ex[m]
            if kind == "int3":
                a["Aq"], a["Bq"] = synth.sample_factor_codes(cfg, e, m)
                a["A"] = a["B"] = None
            elif kind == "bucket":
                a["rank"] = r = bucket[(3 * e + 2 * m) % len(bucket)]
                a["A"] = np.ascontiguousarray(a["A"][:, :r]) if r else None
                a["B"] = np.ascontiguousarray(a["B"][:r]) if r else None
    x_bits = synth.make_tokens(cfg)
    x = amd.bf16_tensor(x_bits)
    ref = fixtures.oracle_forward(cfg, layer, x_bits)
    assert (np.diff(ref["perm"]["offsets"])[:experts - busy] == 0).all()
    Lr, Ls = amd.Layer.from_config(cfg), amd.Layer.from_config(cfg, residency=amd.STAGED)
    Lr.load(layer); Ls.load(layer)
    out_r = Lr.forward(x).clone()
    assert Lr.stats()["path"] == 0
    out_s = Ls.forward(x).clone()
    torch.cuda.synchronize()
    assert orc.rel_frobenius(_to_np(out_r), ref["out"]) <= TOL
    assert torch.equal(out_r.view(torch.int16), out_s.view(torch.int16))
    Lr.close(); Ls.close()


@pytest.mark.parametrize("experts,top_k,tokens", [
    (32, 2, 32), (32, 2, 33),              # 64 pairs; a 65th
    (16, 2, 64), (16, 3, 43),              # two steps; 129 pairs
    (8, 2, 128), (8, 1, 129), (8, 2, 129), # 256 pairs; three steps; 258 pairs
    (33, 1, 5), (3, 3, 85), (1, 1, 256),   # many experts; every token has every expert; one expert
])
def test_forward_of_few_pairs_groups_them_as_permute_does(amd, experts, top_k, tokens):
    """forward() groups few pairs by ballots in the launch that prepares the activations, permute() by the histogram: sizes on both
    sides of the line between them, against the oracle (bf16 rounding: TOL) and the four calls (which may round the expert rows to
    bf16 once more, 2^-9)."""
    cfg = configs.TINY.with_(n_experts=experts, top_k=top_k, top_n=min(top_k, 2), tokens=tokens, ffn=128, rank=16, name=f"few_E{experts}_T{tokens}")
    layer = fixtures.sample_layer(cfg)
    x_bits = synth.make_tokens(cfg)
    x = amd.bf16_tensor(x_bits)
    ref = fixtures.oracle_forward(cfg, layer, x_bits)
    L = amd.Layer.from_config(cfg)
    L.load(layer)
    idx, w = L.route(x)
    counts, offsets, row_pair, pair_row, comp = L.permute(idx)
    for g, key in zip((counts, offsets, row_pair, pair_row, comp), ("counts", "offsets", "row_pair", "pair_row", "comp_counts")):
        np.testing.assert_array_equal(_to_np(g), ref["perm"][key], err_msg=key)
    four = L.combine(L.expert_ffn(x, offsets, row_pair), w, pair_row, x).clone()
    out = L.forward(x)
    assert orc.rel_frobenius(_to_np(out), ref["out"]) <= TOL
    assert orc.rel_frobenius(_to_np(out), _to_np(four)) <= 2.5e-3
    L.close()


@pytest.mark.parametrize("experts,top_k,tokens", [
    (32, 2, 32), (32, 2, 33), (16, 2, 64), (16, 3, 43), (8, 2, 128), (8, 1, 129), (8, 2, 129), (33, 1, 5),      # beyond the line
    (12, 2, 32), (12, 2, 33), (13, 2, 3),  # the most experts, 64 pairs and 66; an expert too many
    (6, 2, 64), (6, 3, 43), (4, 2, 96),    # 128 pairs and 129; three steps
    (3, 3, 85), (3, 2, 129), (1, 1, 256),  # 255 pairs, every token has every expert; 258 pairs; one expert
    (16, 3, 1), (8, 2, 2), (5, 4, 3),      # routed by the launch that groups them
])
def test_forward_leaves_the_arrays_of_permute(amd, experts, top_k, tokens):
    """The five arrays of the grouping that forward() leaves in the workspace are the oracle's, as permute()'s are, on both sides of the line
    between the ballots of the launch that prepares the activations and the histogram."""
    import torch
    cfg = configs.TINY.with_(n_experts=experts, top_k=top_k, top_n=min(top_k, 2), tokens=tokens, ffn=128, rank=16, name=f"few_E{experts}_T{tokens}")
    layer = fixtures.sample_layer(cfg)
    x_bits = synth.make_tokens(cfg)
    x = amd.bf16_tensor(x_bits)
    ref = fixtures.oracle_forward(cfg, layer, x_bits)
    L = amd.Layer.from_config(cfg)
    L.load(layer)
    ws = L.workspace(tokens)
    ws.fill_(0xa5)
    out = L.forward(x)
    torch.cuda.synchronize()
    left, at = ws.cpu().numpy().tobytes(), 0
    for key in ("counts", "offsets", "comp_counts", "row_pair", "pair_row"):
        want = np.asarray(ref["perm"][key]).astype(np.int32).tobytes()
        while at < len(left) and left[at:at + len(want)] != want:
            at += 256                          # (the workspace's arrays start at multiples of 256 bytes, in this order)
        assert at < len(left), f"{key} is not in the workspace"
        at += 256
    assert orc.rel_frobenius(_to_np(out), ref["out"]) <= TOL
    L.close()


@pytest.mark.parametrize("hidden,rank,tokens,experts,top_k,kind", [
    (256, 8, 16, 8, 1, "same"),            # one pass of 16 tokens, one factor tile, as many experts as the rule takes
    (320, 40, 17, 3, 2, "int3"),           # one token in the second pass, an odd number of factor tiles
    (4096, 128, 64, 8, 2, "same"),         # the largest batch and rank (too many blocks: of the routed rows)
    (1088, 64, 49, 16, 2, "bucket"),       # more passes than the grid has (of the routed rows); ranks that differ
    (4096, 32, 64, 8, 2, "int3"),          # the largest batch, four passes of 16 side by side
    (2048, 128, 64, 4, 1, "same"),         # the largest rank, two passes of 32
    (2112, 64, 49, 6, 1, "bucket"),        # two passes of 32, one token in the last half; ranks that differ
    (1024, 24, 32, 32, 4, "same"),         # as many experts as the rule takes, one pass of 32, an odd number of factor tiles
])
def test_x_a13_of_every_token(amd, hidden, rank, tokens, experts, top_k, kind):
    """(x A1 | x A3) of small decode batches is made for every token and expert beside the grouping (where that is few
    blocks): passes, factor
    tiles and tokens at which its indices change, against the oracle and, bit for bit, against a staged layer (whose
    factors arrive later: there the products are made of the routed rows)."""
    import torch
    bucket = (64, 0, 16, 40, 0, 8, 64)
    cfg = configs.TINY.with_(hidden=hidden, ffn=128, n_experts=experts, top_k=top_k, rank=rank, tokens=tokens, bits=2,
                             name=f"x_a13_{kind}_T{tokens}_r{rank}")
    layer = fixtures.sample_layer(cfg)
    for e, ex in enumerate(layer["experts"]):
        for m in (0, 1, 2):
            a = ex[m]
            if kind == "int3":
                a["Aq"], a["Bq"] = synth.sample_factor_codes(cfg, e, m)
                a["A"] = a["B"] = None
            elif kind == "bucket":
                a["rank"] = r = bucket[(3 * e + 2 * m) % len(bucket)]
                a["A"] = np.ascontiguousarray(a["A"][:, :r]) if r else None
                a["B"] = np.ascontiguousarray(a["B"][:r]) if r else None
    x_bits = synth.make_tokens(cfg)
    x = amd.bf16_tensor(x_bits)
    ref = fixtures.oracle_forward(cfg, layer, x_bits)
    Lr = amd.Layer.from_config(cfg)
    Ls = amd.Layer.from_config(cfg, residency=amd.STAGED)
    Lr.load(layer); Ls.load(layer)
    out_r = Lr.forward(x).clone()
    out_s = Ls.forward(x).clone()
    torch.cuda.synchronize()
    err = orc.rel_frobenius(_to_np(out_r), ref["out"])
    print(f"\n[{cfg.name}] out rel err {err:.2e}", flush=True)
    assert err <= TOL
    assert torch.equal(out_r.view(torch.int16), out_s.view(torch.int16))
    Lr.close(); Ls.close()


@pytest.mark.parametrize("hidden,ffn,bits,rank,top_n,kind", [
    (320, 576, 2, 24, 1, "same"),          # odd numbers of k-steps in both products, two n-tiles of W2 per wavefront
    (2560, 512, 3, 8, 1, "int3"),          # four n-tiles of W2; two k-steps
    (512, 256, 4, 40, 1, "same"),          # one k-step in W2, 4 bits (a second slot for two row pairs only)
    (4096, 1024, 3, 0, 0, "same"),         # an expert's weights beyond half an L2: column blocks dealt over the XCDs
])
def test_grouped_gemm_chunks_of_every_length(amd, hidden, ffn, bits, rank, top_n, kind):
    """Rows per expert given by hand: none, one, one short of a fragment or a chunk, exactly one, one more, several.  The
    grouped GEMM finds its chunks by length and takes the k loop of their number of row pairs; every row against the oracle."""
    import torch
    counts = [0, 1, 31, 32, 33, 64, 65, 96, 97, 127, 128, 129, 256, 353, 512, 0, 288]
    E, T = len(counts), sum(counts)
    cfg = configs.TINY.with_(hidden=hidden, ffn=ffn, n_experts=E, top_k=1, top_n=top_n, rank=rank, tokens=T, bits=bits, name=f"chunks_{bits}b_{hidden}")
    layer = fixtures.sample_layer(cfg)
    if kind == "int3":
        for e, ex in enumerate(layer["experts"]):
            for m in (0, 1, 2):
                ex[m]["Aq"], ex[m]["Bq"] = synth.sample_factor_codes(cfg, e, m)
                ex[m]["A"] = ex[m]["B"] = None
    idx = np.random.default_rng(7).permutation(np.repeat(np.arange(E, dtype=np.int32), counts)).reshape(T, 1)
    x_bits = synth.make_tokens(cfg)
    perm = orc.permute(idx, E, cfg.top_n)
    want = orc.expert_ffn(x_bits, perm, layer["experts"], 1, cfg.top_n, cfg.group)
    L = amd.Layer.from_config(cfg)
    L.load(layer)
    x = amd.bf16_tensor(x_bits)
    got_counts, offsets, row_pair, _, _ = L.permute(torch.from_numpy(idx).cuda())
    assert _to_np(got_counts).tolist() == counts
    y = _to_np(L.expert_ffn(x, offsets, row_pair))
    assert L.stats()["path"] == 3
    worst = max(orc.rel_frobenius(y[a:b], want[a:b]) for a, b in zip(perm["offsets"][:-1], perm["offsets"][1:]) if b > a)
    print(f"\n[{cfg.name}] path {L.stats()['path']}, rel err {orc.rel_frobenius(y, want):.2e}, worst expert {worst:.2e}", flush=True)
    assert orc.rel_frobenius(y, want) <= TOL and worst <= 2 * TOL      # (an expert of one row has no average over rows)
    L.close()


def test_residency_does_not_change_bits_where_the_workspace_is_tight(amd):
    """FFN width 960, hidden 256, 16 experts: the part sums of (h A2) and (x A1 | x A3) of every token do not fit the same room
    together.  Which of them is taken must not decide the order of any sum: resident and staged layers, bit for bit."""
    import torch
    cfg = configs.TINY.with_(hidden=256, ffn=960, n_experts=16, top_k=2, rank=32, tokens=16, bits=2, name="tight_room")
    layer = fixtures.sample_layer(cfg)
    Lr = amd.Layer.from_config(cfg)
    Ls = amd.Layer.from_config(cfg, residency=amd.STAGED)
    Lr.load(layer); Ls.load(layer)
    for seed in range(100):
        x = amd.bf16_tensor(synth.make_tokens(cfg.with_(seed=3000 + seed)))
        out_r = Lr.forward(x).clone()
        out_s = Ls.forward(x).clone()
        assert torch.equal(out_r.view(torch.int16), out_s.view(torch.int16)), seed
    Lr.close(); Ls.close()
