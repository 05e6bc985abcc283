"""What (x A) and (h A) of the grouped-GEMM flavour cost where their work differs from one layer to the
next, as ratios of two stage times of one process (the smallest of several runs each): a launch that
does work it need not do shows as a ratio near the one of the two shapes."""
import numpy as np
import pytest

from workload import configs, synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def amd():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    import paper_2512_17073_amd as amd
    amd.lib()
    return amd


def _stage_us(amd, cfg, stage, own_rank=None, int3=False):
    """Smallest time of `stage` over twelve forwards of a layer whose pairs all have rank own_rank (the layer's
    rank if None); every expert stores the same artefacts."""
    import torch
    r = cfg.rank if own_rank is None else own_rank
    one = {m: synth.sample_artifacts(cfg.with_(rank=r), 0, m) for m in (0, 1, 2)}
    L = amd.Layer.from_config(cfg)
    L.set_gate(*synth.make_gate(cfg))
    q3 = {m: synth.sample_factor_codes(cfg, 0, m) for m in (0, 1, 2)} if int3 else None
    for e in range(cfg.n_experts):
        for m, a in one.items():
            if int3:
                L.set_expert(e, m, a["codes"], a["scale"], a["zero"], None, None, 0)
                L.set_expert_factors_quantized(e, m, r, *q3[m])
            else:
                L.set_expert(e, m, a["codes"], a["scale"], a["zero"], a["A"], a["B"], r)
    x = amd.bf16_tensor(synth.make_tokens(cfg))
    L.profile_enable(True)
    best = np.inf
    for i in range(14):
        L.forward(x)
        torch.cuda.synchronize()
        if i >= 2:
            best = min(best, L.profile_read()[stage] * 1e3)
    L.close()
    print(f"\n[{cfg.name}] {stage} {best:.1f} us", flush=True)
    return best


WIDE = configs.QWEN3.with_(n_experts=64, tokens=2048, ffn=512, zipf_s=0.0)


def test_tiles_past_a_pairs_own_rank_cost_little(amd):
    """A layer whose largest rank is 1024 while its pairs have 16 (Section 3.1 allocates ranks far apart):
    computing the empty factor tiles takes as long as a layer with all pairs at 1024, leaving
    them out a quarter of that."""
    full = _stage_us(amd, WIDE.with_(rank=1024, name="all_1024"), "xa13")
    dead = _stage_us(amd, WIDE.with_(rank=1024, name="largest_1024_own_16"), "xa13", own_rank=16)
    assert dead < 0.6 * full


def test_int3_pairs_cost_little_more_than_fp16_ones(amd):
    """(x A1 | x A3) of pairs held at 3 bits beside the same layer with fp16 pairs: a quarter of the
    factor bytes and some dequantizing.  A block that holds more operands than its registers and spills them takes
    more than twice as long."""
    cfg = configs.MIXTRAL_DECODE.with_(ffn=512, rank=64, tokens=1024, bits=3)
    plain = _stage_us(amd, cfg.with_(name="fp16_pairs"), "xa13")
    packed = _stage_us(amd, cfg.with_(name="int3_pairs"), "xa13", int3=True)
    assert packed < 1.5 * plain


def test_large_ranks_read_the_rows_a_few_times_only(amd):
    """Rank 1024 against rank 64, both at their own size: sixteen times the factor tiles.  With the rows read
    again for every four tiles that costs ten times the time or more, with the rows staged once per 32 tiles
    about six times."""
    small = _stage_us(amd, WIDE.with_(rank=64, tokens=4096, name="rank_64"), "xa13")
    large = _stage_us(amd, WIDE.with_(rank=1024, tokens=4096, name="rank_1024"), "xa13")
    assert large < 8.5 * small


def test_a_long_k_with_several_tiles_does_not_gather_pieces(amd):
    """(h A2) over K = 14336 at rank 256 against rank 16: 2.4 times with the rows staged, 3.7 times with each row's
    16-byte pieces gathered again for every four tiles (82 and 127 us against 34); the line lies between."""
    cfg = configs.MIXTRAL_PREFILL.with_(hidden=1024, tokens=2048)
    small = _stage_us(amd, cfg.with_(rank=16, name="long_k_rank_16"), "xa2")
    large = _stage_us(amd, cfg.with_(rank=256, name="long_k_rank_256"), "xa2")
    assert large < 3.0 * small
