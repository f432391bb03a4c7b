"""The prefill GEMM's tile shapes in the model: a batch whose GEMMs run 256 x 256 tiles and one environment of it, whose
GEMMs run smaller tiles, or are cut by rows or columns into both, give the same bits through the forward's epilogues
(residual in place, SwiGLU, RoPE + KV append); and a gradient whose products are cut (residual from one buffer to another,
SwiGLU with kept pre-activations, the input gradients' plain stores) equals what other routes give."""
import ctypes

import numpy as np
import pytest
import torch

from gpu_util import Setup
from paper_2505_18719_amd import inputs, vla

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,heads,ffn,batch", [(256, 4, 688, 40), (1024, 8, 2752, 20), (1024, 8, 2752, 96), (2048, 16, 5496, 48),
                                               (2048, 16, 5496, 64)])
def test_one_environment_matches_the_batch(d, heads, ffn, batch):
    cfg = inputs.TINY.replace(name="shapes", d_model=d, n_heads=heads, d_ffn=ffn, batch=batch, prompt_min=0,
                              prompt_max=57)
    S = Setup(cfg, seed=31)
    lens = np.random.default_rng(31).integers(0, 58, size=batch).astype(np.int32)
    lens[:3] = [57, 0, 33]
    inp, dev = S.inputs(seed=31, prompt_lens=lens)
    acts = torch.from_numpy(inputs.stored_actions(cfg, batch, seed=31)).cuda()
    full = S.model.token_logprobs(dev["vis"], dev["ids"], lens, acts, 1.5)
    S.model.prefill(dev["vis"], dev["ids"], lens)
    dec = {k: v.clone() for k, v in S.model.decode_actions(dev["gumbel"], 1.5).items()}
    for b in (0, 1, 2, batch - 1):
        off, n = int(lens[:b].sum()), int(lens[b])
        ids, vis = dev["ids"][off:off + n].contiguous(), dev["vis"][b:b + 1].contiguous()
        one = S.model.token_logprobs(vis, ids, lens[b:b + 1], acts[b:b + 1].contiguous(), 1.5)
        for k in one:
            assert torch.equal(one[k][0], full[k][b]), (b, k)
        S.model.prefill(vis, ids, lens[b:b + 1])
        got = S.model.decode_actions(dev["gumbel"][b:b + 1].contiguous(), 1.5)
        for k in got:
            assert torch.equal(got[k][0], dec[k][b]), (b, k)
    S.model.close()


class _GemmPlan(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int) for n in ("first", "rest", "rows", "cols")]


def test_gradients_through_cut_products():
    """Both training modes of a batch whose O, down, gate/up, QKV and input-gradient products are cut (the plan says so):
    the log-probs are the bits of the scoring pass, whose residual stream is updated in place; keeping the gate/up
    pre-activations gives the bits of recomputing them through another epilogue; and the gradients are the sums of those of
    quarter batches, whose products are not cut so.  Each row's part is the same bits up to the power of two of 1 / n, so
    only the order of the fp32 sums over the M rows differs (8 M 2^-24 of the norm)."""
    B, rank = 32, 16
    cfg = inputs.TINY.replace(name="cut_grads", n_layers=2, d_model=2048, n_heads=16, d_ffn=5504, n_visual=256, batch=B,
                              prompt_min=0, prompt_max=40)
    S = Setup(cfg, seed=61)
    inp, dev = S.inputs(seed=61)
    lens = inp.prompt_lens
    M, d, F = int(B * (256 + cfg.n_actions) + lens.sum()), cfg.d_model, cfg.d_ffn
    plan = vla.load_library()["_ZN3vla9gemm_planEiiiiNS_12GemmEpilogueE"]
    plan.restype, plan.argtypes = _GemmPlan, [ctypes.c_int] * 5
    cus = torch.cuda.get_device_properties(0).multi_processor_count // 8 * 8
    cuts = [plan(M, n, k, cus, epi) for n, k, epi in ((d, d, 1), (d, F, 1), (3 * d, d, 3), (2 * F, d, 4), (d, 3 * d, 0))]
    assert all(p.rows + p.cols > 0 for p in cuts), [(p.first, p.rows, p.cols) for p in cuts]
    assert any(p.rows for p in cuts[:2]) and any(p.cols for p in cuts)
    ad = inputs.make_lora(cfg, rank, seed=61, device="cuda")
    acts = torch.from_numpy(inputs.stored_actions(cfg, B, seed=61)).cuda()
    tf = S.model.token_logprobs(dev["vis"], dev["ids"], lens, acts, 1.5)
    rng = np.random.default_rng(61)
    old = tf["logp"] + 0.01 * torch.from_numpy(rng.normal(size=(B, cfg.n_actions)).astype(np.float32)).cuda()
    adv = torch.from_numpy(rng.normal(size=B).astype(np.float32)).cuda()
    off = np.concatenate([[0], np.cumsum(lens)])

    def grads(a, b, mode):
        return S.model.ppo_lora_grads(dev["vis"][a:b].contiguous(), dev["ids"][off[a]:off[b]].contiguous(), lens[a:b],
                                      acts[a:b].contiguous(), old[a:b].contiguous(), adv[a:b].contiguous(), 0.2, 1.5, ad, 0.5,
                                      mode=mode)

    _, logp, keep = grads(0, B, vla.TRAIN_KEEP)
    assert torch.equal(logp, tf["logp"])
    sums = [{k: [torch.zeros_like(g, dtype=torch.float64) for g in ab] for k, ab in layer.items()} for layer in keep]
    for q in range(4):
        part = grads(q * B // 4, (q + 1) * B // 4, vla.TRAIN_KEEP)[2]
        for s, p in zip(sums, part):
            for k in s:
                for t, g in zip(s[k], p[k]):
                    t += g.double() / 4
    _, logp2, again = grads(0, B, vla.TRAIN_RECOMPUTE)
    assert torch.equal(logp2, logp)
    for li, layer in enumerate(keep):
        for k, ab in layer.items():
            for f in range(2):
                assert torch.equal(ab[f], again[li][k][f]), (li, k, f)
                err = (ab[f].double() - sums[li][k][f]).norm() / sums[li][k][f].norm()
                assert err <= 8 * M * 2.0 ** -24, (li, k, f, float(err))
    S.model.close()
