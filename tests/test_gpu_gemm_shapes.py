"""The prefill GEMM's tile shapes in the model: a batch whose GEMMs run 256 x 256 tiles and one environment of it,
whose GEMMs run smaller tiles, or are cut by rows or columns into both, give the same bits through every epilogue (residual, SwiGLU, RoPE + KV append, and the
kept pre-activations of the gradient's forward)."""
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
