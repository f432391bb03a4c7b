"""The persistent decode layer kernel (one cooperative launch per decoder
layer and decode step, grid barriers between its phases) against the
per-kernel decode path: the same inputs give the same bits, at tiny, mid and
7B width, with one and with several 128-row decode chunks, and no barrier
wait times out."""
import numpy as np
import pytest
import torch

from gpu_util import Setup, log
from paper_2505_18719_amd import inputs

pytestmark = pytest.mark.gpu

FLAG_SYNC_TIMEOUT = 4


def _both_paths(S, inp, dev, T):
    outs = []
    for path in (0, 1):
        S.model.debug_decode_path(path)
        S.model.prefill(dev["vis"], dev["ids"], inp.prompt_lens)
        out = S.model.decode_actions(dev["gumbel"], T)
        torch.cuda.synchronize()
        outs.append({k: v.clone() for k, v in out.items()})
        assert S.model.read_flags() & FLAG_SYNC_TIMEOUT == 0
    S.model.debug_decode_path(0)
    return outs


@pytest.mark.parametrize("name", ["tiny_ragged", "mid", "7b_width_2l_b64", "tiny_b200"])
def test_persistent_decode_matches_the_per_kernel_path_bitwise(name):
    if name == "tiny_ragged":
        cfg, T, lens = inputs.TINY.replace(name=name, batch=5, prompt_min=0, prompt_max=40), 1.5, [0, 40, 7, 33, 16]
    elif name == "mid":
        cfg, T, lens = inputs.MID, 1.0, None
    elif name == "7b_width_2l_b64":
        cfg, T, lens = inputs.L7B_B64.replace(n_layers=2), 1.5, None
    else:
        cfg, T, lens = inputs.TINY.replace(name=name, batch=200, prompt_min=0, prompt_max=57), 1.5, None
    S = Setup(cfg, seed=11)
    inp, dev = S.inputs(seed=11, prompt_lens=lens)
    log(f"[decode paths {name}] batch {inp.batch}")
    ref, got = _both_paths(S, inp, dev, T)
    for k in ref:
        same = torch.equal(ref[k], got[k])
        if not same:
            d = (ref[k].double() - got[k].double()).abs().max().item()
            log(f"[decode paths {name}] {k} differs, max |d| {d:.3e}")
        assert same, k
    log(f"[decode paths {name}] tokens, log-probs, entropies, logits: identical bits")
    S.model.close()


@pytest.mark.parametrize("head_dim", [64, 128])
def test_decode_attention_variants_give_the_same_bits(head_dim):
    """An environment decodes to the same bits alone, among 30 and among 128 of 16 heads: the decode attention's variants
    for at most one workgroup per CU, at most four, and more.  Sequences end at the first and last slot of a page and at
    the longest length."""
    lens = np.array([0, 57, 9, 16, 15, 1, 40, 33, 25, 56] + [(7 * i) % 58 for i in range(118)], dtype=np.int32)
    cfg = inputs.TINY.replace(name=f"hd{head_dim}", n_layers=1, d_model=16 * head_dim, n_heads=16, batch=128,
                              prompt_min=0, prompt_max=57)
    S = Setup(cfg, seed=13)
    inp, dev = S.inputs(seed=13, prompt_lens=lens)
    off = np.concatenate([[0], np.cumsum(inp.prompt_lens)])

    def run(a, b):
        S.model.prefill(dev["vis"][a:b].contiguous(), dev["ids"][off[a]:off[b]].contiguous(), inp.prompt_lens[a:b])
        out = S.model.decode_actions(dev["gumbel"][a:b].contiguous(), 1.5)
        torch.cuda.synchronize()
        return {k: v.clone() for k, v in out.items()}

    full, some = run(0, 128), run(0, 30)
    for k in full:
        assert torch.equal(full[k][:30], some[k]), k
    for b in range(10):
        one = run(b, b + 1)
        for k in full:
            assert torch.equal(full[k][b], one[k][0]), (k, b)
    S.model.close()


@pytest.mark.parametrize("d,ffn,layers", [(2048, 5504, 4), (2560, 8192, 2)])
def test_weights_past_the_caches_give_the_same_bits(d, ffn, layers):
    """Weights above 256 MB with products on both sides of 28 and 48 MB: environments decode to the bits that they get
    among 65 (every product through the caches) at 1, 16 and 32 rows (past them from 28 MB on) and at 33 and 64 (from 48)."""
    cfg = inputs.TINY.replace(name=f"past{d}", n_layers=layers, d_model=d, n_heads=d // 64, d_ffn=ffn, n_visual=16, batch=65,
                              prompt_min=0, prompt_max=20)
    fp = (ffn + 255) // 256 * 256
    mb = sorted(2 * n / 2 ** 20 for n in (3 * d * d, d * d, 2 * fp * d, fp * d))
    assert layers * sum(mb) > 256 and mb[0] < 28 and any(28 <= m < 48 for m in mb)
    S = Setup(cfg, seed=17)
    inp, dev = S.inputs(seed=17)
    off = np.concatenate([[0], np.cumsum(inp.prompt_lens)])

    def run(n):
        S.model.prefill(dev["vis"][:n].contiguous(), dev["ids"][:off[n]].contiguous(), inp.prompt_lens[:n])
        out = S.model.decode_actions(dev["gumbel"][:n].contiguous(), 1.5)
        torch.cuda.synchronize()
        return {k: v.clone() for k, v in out.items()}

    full = run(65)
    for n in (1, 16, 32, 33, 64):
        got = run(n)
        for k in full:
            assert torch.equal(full[k][:n], got[k]), (k, n)
    S.model.close()


def test_persistent_decode_repeats_bit_exactly():
    S = Setup(inputs.L7B_B64.replace(n_layers=2), seed=12)
    S.model.debug_decode_path(1)
    inp, dev = S.inputs(seed=12)
    outs = []
    for _ in range(3):
        S.model.prefill(dev["vis"], dev["ids"], inp.prompt_lens)
        out = S.model.decode_actions(dev["gumbel"], 1.5)
        torch.cuda.synchronize()
        outs.append({k: v.clone() for k, v in out.items()})
    for o in outs[1:]:
        for k in o:
            assert torch.equal(o[k], outs[0][k]), k
    assert S.model.read_flags() == 0
    S.model.close()
