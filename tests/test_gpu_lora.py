"""Parity of the LoRA merge (Sec. 3.3, Rollout Phase: the updated LoRA weights
are merged with the original checkpoint before the rollout) with the CPU
oracle: the packed weights the rollout reads, read back and unpacked on the
host from their documented layout, and a rollout of the merged policy."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import LOGIT_TOL, LOGP_TOL, Setup, compare_rollout, log
from paper_2505_18719_amd import inputs

pytestmark = pytest.mark.gpu

PROJ = ("wq", "wk", "wv", "wo", "wgate", "wup", "wdown")
SCALE = 0.5   # alpha / rank of the adapter


# ---------------------------------------------------------------- layouts
def _fp(d_ffn):
    return (d_ffn + 255) // 256 * 256


def _frag_gather(buf, rows, K):
    """Rows `rows` of a frag-layout bf16 matrix with K columns (vla_debug.h):
    element (r, k) sits at ((((r//16) (K/32 + 1) + k//32) * 64) + r%16 + 16 ((k%32)//8)) * 8 + k%8."""
    KB = K // 32 + 1
    r = np.asarray(rows)[:, None]
    k = np.arange(K)[None, :]
    idx = ((((r >> 4) * KB + (k >> 5)) << 6) + (r & 15) + (((k & 31) >> 3) << 4)) * 8 + (k & 7)
    raw = buf.view(torch.int16).cpu().numpy()[idx]
    return torch.from_numpy(raw).view(torch.bfloat16).double().numpy()


def _packed_source(cfg, which, r):
    """(projection key, source row or -1 for a zero row) of packed row r."""
    d, hd, F = cfg.d_model, cfg.head_dim, cfg.d_ffn
    if which == 5:
        part, rr = divmod(r, d)
        if part == 2:
            return "wv", rr
        head, p = divmod(rr, hd)
        blk, c = divmod(p, 64)
        return ("wq", "wk")[part], head * hd + (32 * blk + c if c < 32 else hd // 2 + 32 * blk + c - 32)
    if which == 6:
        return "wo", r
    if which == 7:
        j = 32 * (r // 64) + r % 32
        return ("wgate" if r % 64 < 32 else "wup"), (j if j < F else -1)
    return "wdown", r


def _packed_shape(cfg, which):
    d, Fp = cfg.d_model, _fp(cfg.d_ffn)
    return {5: (3 * d, d), 6: (d, d), 7: (2 * Fp, d), 8: (d, Fp)}[which]


def _read_packed(model, cfg, which, layer):
    R, K = _packed_shape(cfg, which)
    n = (R + 15) // 16 * (K // 32 + 1) * 512
    buf = torch.empty(n, dtype=torch.bfloat16, device="cuda")
    model.debug_read(which, layer, buf)
    torch.cuda.synchronize()
    return buf


def _check_packed(cfg, buf, which, rows, w0_layer, adapters, scale, label):
    """Packed rows `rows` against the oracle merge of the source rows: exact,
    except where the float64 value v lies within the fp32 accumulation error
    e of the rank sum from a bf16 rounding boundary; there the result must be
    a bf16 value in [bf16(v - e), bf16(v + e)] (where W0 and the update nearly
    cancel, that interval spans several bf16 steps)."""
    R, K = _packed_shape(cfg, which)
    got = _frag_gather(buf, rows, K)
    n_exact = n_edge = 0
    for i, r in enumerate(rows):
        key, j = _packed_source(cfg, which, int(r))
        exp = np.zeros(K)
        if j >= 0:
            w0 = oracle.to_f64(w0_layer[key][j:j + 1])
            ncol = w0.shape[1]
            if adapters is not None and key in adapters:
                a, b = oracle.to_f64(adapters[key][0]), oracle.to_f64(adapters[key][1][j:j + 1])
                v = w0 + scale * (b @ a)
                err = 2.0 ** -24 * (a.shape[0] + 4) * (np.abs(w0) + abs(scale) * (np.abs(b) @ np.abs(a)))
                lo, hi = oracle.bf16_round(v - err), oracle.bf16_round(v + err)
                m = oracle.lora_merge(w0_layer[key][j:j + 1], adapters[key][0], adapters[key][1][j:j + 1], scale)
                g = got[i, :ncol]
                ok = (g == m) | ((g >= lo) & (g <= hi))  # a rounding of some value within the fp32 error
                if not ok.all():
                    bad = np.where(~ok)[1][:3]
                    detail = [(int(c), float(v[0, c]), float(m[0, c]), float(g[c]), float(lo[0, c]), float(hi[0, c]),
                               float(err[0, c]), float(w0[0, c]), float((b @ a)[0, c])) for c in bad]
                    raise AssertionError(f"{label} {key} row {j}: (col, exact, oracle, gpu, lo, hi, err, w0, BA) {detail}")
                n_exact += int((g == m).sum())
                n_edge += int((g != m).sum())
                exp = None
            else:
                exp[:ncol] = w0[0]
        if exp is not None:
            assert np.array_equal(got[i], exp), (label, key, j)
        elif got.shape[1] > w0.shape[1]:
            assert not got[i, w0.shape[1]:].any(), (label, key, "padding columns")
    log(f"[{label}] rows={len(rows)} merged elements exact={n_exact} rounding-boundary neighbours={n_edge}")
    return n_exact, n_edge


def _same_bits(x, y):
    """Bitwise equality (torch.equal on bf16 compares values, and NaN != NaN)."""
    return torch.equal(x.view(torch.int16), y.view(torch.int16))


def _assert_same_packed(cfg, which, got, exp, msg):
    """Bitwise equality of two packed buffers; on a mismatch, name the first
    differing elements as (row, column) or as a spare block."""
    if _same_bits(got, exp):
        return
    _, K = _packed_shape(cfg, which)
    kb = K // 32 + 1
    idx = torch.nonzero(got.view(torch.int16) != exp.view(torch.int16)).flatten().cpu().numpy()
    where = []
    for i in idx[:6]:
        blk, lane_e = divmod(int(i), 512)
        rb, kblk = divmod(blk, kb)
        lane, e = divmod(lane_e, 8)
        where.append("spare" if kblk == K // 32 else (16 * rb + lane % 16, 32 * kblk + 8 * (lane // 16) + e))
    raise AssertionError(f"{msg}: {len(idx)} of {got.numel()} elements differ, first at {where}")


# ---------------------------------------------------------------- tests
@pytest.fixture(scope="module")
def tiny():
    return Setup(inputs.TINY, seed=0)


def _merge_all(S, adapters, scale, layers):
    for li, ad in zip(layers, adapters):
        for k in PROJ:
            a, b = ad[k]
            S.model.lora_merge(li, k, S.w["layers"][li][k], a, b, scale)


def test_packed_weights_spare_blocks_are_zero(tiny):
    """Every byte of a packed weight is defined: the spare block that ends each
    16-row block is zero after create (and a merge never writes it)."""
    S, cfg = tiny, inputs.TINY
    for which in (5, 6, 7, 8):
        R, K = _packed_shape(cfg, which)
        kb = K // 32 + 1
        blocks = _read_packed(S.model, cfg, which, cfg.n_layers - 1).view(torch.int16).view(-1, kb, 512)
        assert blocks.shape[0] == (R + 15) // 16
        assert not blocks[:, kb - 1].any(), which


@pytest.mark.parametrize("rank", [8, 32])
def test_lora_merge_packed_weights_match_oracle(tiny, rank):
    S, cfg = tiny, inputs.TINY
    before0 = {w: _read_packed(S.model, cfg, w, 0).clone() for w in (5, 6, 7, 8)}
    ad = inputs.make_lora(cfg, rank, seed=rank, device="cuda", layers=[1])
    _merge_all(S, ad, SCALE, [1])
    adc = {k: (a.cpu(), b.cpu()) for k, (a, b) in ad[0].items()}
    edge = 0
    for which in (5, 6, 7, 8):
        buf = _read_packed(S.model, cfg, which, 1)
        R, _ = _packed_shape(cfg, which)
        edge += _check_packed(cfg, buf, which, range(R), S.wc["layers"][1], adc, SCALE, f"tiny r{rank} w{which}")[1]
        _assert_same_packed(cfg, which, _read_packed(S.model, cfg, which, 0), before0[which], "layer 0 must be untouched")
    assert edge <= 8
    # restore the checkpoint for the other tests of the module
    _merge_all(S, [{k: (a, torch.zeros_like(b)) for k, (a, b) in ad[0].items()}], SCALE, [1])


@pytest.mark.parametrize("key", ["wgate", "wup"])
def test_lora_merge_of_one_mlp_part_leaves_the_other_rows(tiny, key):
    """The packed [gate; up] weight interleaves the two projections in 32-row
    halves; merging one of them computes and writes only its own rows (checked
    against the oracle), the other part's rows keep their bits, and a zero
    update restores the whole buffer."""
    S, cfg = tiny, inputs.TINY
    before = _read_packed(S.model, cfg, 7, 0).clone()
    a, b = inputs.make_lora(cfg, 16, seed=11, device="cuda", layers=[0])[0][key]
    S.model.lora_merge(0, key, S.w["layers"][0][key], a, b, SCALE)
    buf = _read_packed(S.model, cfg, 7, 0)
    R, K = _packed_shape(cfg, 7)
    mine = [r for r in range(R) if _packed_source(cfg, 7, r)[0] == key]
    other = [r for r in range(R) if _packed_source(cfg, 7, r)[0] != key]
    _check_packed(cfg, buf, 7, mine, S.wc["layers"][0], {key: (a.cpu(), b.cpu())}, SCALE, f"tiny {key} alone")
    assert np.array_equal(_frag_gather(buf, other, K), _frag_gather(before, other, K)), "the other part's rows changed"
    S.model.lora_merge(0, key, S.w["layers"][0][key], a, torch.zeros_like(b), SCALE)
    _assert_same_packed(cfg, 7, _read_packed(S.model, cfg, 7, 0), before, "a zero update must restore the packing")


def test_lora_merge_layer_gives_the_bits_of_the_separate_merges(tiny):
    """vla_lora_merge_layer (every projection of a layer in one launch) leaves
    the packed weights of the seven separate vla_lora_merge calls, bit for
    bit; a projection without an adapter in the call keeps its bits."""
    S, cfg = tiny, inputs.TINY
    before = {w: _read_packed(S.model, cfg, w, 1).clone() for w in (5, 6, 7, 8)}
    ad = inputs.make_lora(cfg, 24, seed=13, device="cuda", layers=[1])
    _merge_all(S, ad, SCALE, [1])
    sep = {w: _read_packed(S.model, cfg, w, 1).clone() for w in (5, 6, 7, 8)}
    zero = {k: (a, torch.zeros_like(b)) for k, (a, b) in ad[0].items()}
    _merge_all(S, [zero], SCALE, [1])
    S.model.lora_merge_layer(1, S.w["layers"][1], ad[0], SCALE)
    for w in (5, 6, 7, 8):
        _assert_same_packed(cfg, w, _read_packed(S.model, cfg, w, 1), sep[w], "one launch per layer")
    # without 'wo' and 'wup' in the call: o keeps the merged bits of the previous call, and
    # after restoring the rest, [gate; up] holds the original up rows and o its merged rows
    S.model.lora_merge_layer(1, S.w["layers"][1], {k: v for k, v in zero.items() if k not in ("wo", "wup")}, SCALE)
    _assert_same_packed(cfg, 6, _read_packed(S.model, cfg, 6, 1), sep[6], "o not in the call")
    _assert_same_packed(cfg, 5, _read_packed(S.model, cfg, 5, 1), before[5], "q, k, v restored")
    _assert_same_packed(cfg, 8, _read_packed(S.model, cfg, 8, 1), before[8], "down restored")
    S.model.lora_merge_layer(1, S.w["layers"][1], zero, SCALE)
    for w in (5, 6, 7, 8):
        _assert_same_packed(cfg, w, _read_packed(S.model, cfg, w, 1), before[w], "a zero update restores the layer")


def test_weights_read_back_in_part():
    """Reads on either side of the size from which a kernel copies, of whole and of odd numbers of 16 bytes, and into an
    unaligned buffer hold the first bytes of the whole read, and nothing past them is written."""
    cfg = inputs.TINY.replace(name="read", n_layers=1, d_model=1024, n_heads=8, d_ffn=2752, batch=1)
    S = Setup(cfg, seed=6, max_batch=1)
    whole = _read_packed(S.model, cfg, 7, 0)
    edge = (8 << 20) // 2
    for n in (1, 8, 12345, edge - 8, edge, edge + 1, edge + 8 * 1024 + 8, whole.numel()):
        for skip in (0, 1):
            buf = torch.full((skip + n + 8,), 7.0, dtype=torch.bfloat16, device="cuda")
            S.model.debug_read(7, 0, buf[skip:skip + n])
            assert _same_bits(buf[skip:skip + n], whole[:n]), (n, skip)
            assert bool((buf[skip + n:] == 7.0).all()) and bool((buf[:skip] == 7.0).all()), (n, skip)
    S.model.close()


@pytest.mark.parametrize("rank", [8, 64])
def test_lora_merge_tile_widths_give_the_same_bits(rank):
    """A layer whose weights are stored past the caches, merged in one launch (128-column tiles at rank 8) and projection by
    projection (64-column tiles): the same bits, and sampled rows as the oracle's.  d_ffn ends inside a tile of either."""
    cfg = inputs.TINY.replace(name="wide", n_layers=1, d_model=2560, n_heads=20, d_ffn=6792, batch=1)
    S = Setup(cfg, seed=5, max_batch=1)
    ad = inputs.make_lora(cfg, rank, seed=5, device="cuda")
    _merge_all(S, ad, SCALE, [0])
    sep = {w: _read_packed(S.model, cfg, w, 0).clone() for w in (5, 6, 7, 8)}
    S.model.lora_merge_layer(0, S.w["layers"][0], {k: (a, torch.zeros_like(b)) for k, (a, b) in ad[0].items()}, SCALE)
    S.model.lora_merge_layer(0, S.w["layers"][0], ad[0], SCALE)
    adc = {k: (a.cpu(), b.cpu()) for k, (a, b) in ad[0].items()}
    for w in (5, 6, 7, 8):
        buf = _read_packed(S.model, cfg, w, 0)
        _assert_same_packed(cfg, w, buf, sep[w], f"rank {rank}")
        R, _ = _packed_shape(cfg, w)
        _check_packed(cfg, buf, w, [0, 31, 32, 63, 64, R // 3, R // 2 + 1, R - 65, R - 1], S.wc["layers"][0], adc, SCALE,
                      f"d 2560 r{rank} w{w}")
    S.model.close()


def test_lora_merge_starts_from_the_original_and_a_zero_update_restores(tiny):
    S, cfg = tiny, inputs.TINY
    packed0 = {w: _read_packed(S.model, cfg, w, 0).clone() for w in (5, 6, 7, 8)}
    ad = inputs.make_lora(cfg, 16, seed=5, device="cuda", layers=[0])
    _merge_all(S, ad, SCALE, [0])
    once = {w: _read_packed(S.model, cfg, w, 0).clone() for w in (5, 6, 7, 8)}
    assert not _same_bits(once[5], packed0[5])
    _merge_all(S, ad, SCALE, [0])  # merging again starts from the original: same bits
    for w in once:
        _assert_same_packed(cfg, w, _read_packed(S.model, cfg, w, 0), once[w], "a second merge must give the same bits")
    zero = [{k: (a, torch.zeros_like(b)) for k, (a, b) in ad[0].items()}]
    _merge_all(S, zero, SCALE, [0])
    for w in packed0:
        _assert_same_packed(cfg, w, _read_packed(S.model, cfg, w, 0), packed0[w], "a zero update must restore the packing")


def test_merged_policy_rollout_matches_oracle(tiny):
    S, cfg = tiny, inputs.TINY
    ad = inputs.make_lora(cfg, 32, seed=7, device="cuda")
    _merge_all(S, ad, SCALE, range(cfg.n_layers))
    try:
        merged = oracle.as_weights(oracle.merge_weights(S.wc, [{k: (a.cpu(), b.cpu()) for k, (a, b) in d.items()}
                                                             for d in ad], SCALE), cfg)
        inp, dev = S.inputs(seed=9)
        S.model.prefill(dev["vis"], dev["ids"], inp.prompt_lens)
        out = S.model.decode_actions(dev["gumbel"], 1.5)
        torch.cuda.synchronize()
        st = compare_rollout(cfg, merged, inp, out, 1.5, label="tiny merged")
        assert st["dlogit"] <= LOGIT_TOL and st["dlogp"] <= LOGP_TOL and st["mismatches"] == 0
        # the merge changed the policy: the unmerged oracle is far from it
        base = compare_rollout(cfg, S.W, inp, out, 1.5, label="tiny merged vs unmerged oracle")
        assert base["dlogit"] > 10 * st["dlogit"]
    finally:
        _merge_all(S, [{k: (a, torch.zeros_like(b)) for k, (a, b) in d.items()} for d in ad], SCALE,
                   range(cfg.n_layers))


def test_lora_merge_errors(tiny):
    from paper_2505_18719_amd.vla import VlaError
    S = tiny
    a, b = inputs.make_lora(inputs.TINY, 16, seed=1, device="cuda", layers=[0])[0]["wq"]
    w0 = S.w["layers"][0]["wq"]
    with pytest.raises(VlaError, match="VLA_EUNSUPPORTED"):
        S.model.lora_merge(0, "wq", w0, a[:12].contiguous(), b[:, :12].contiguous(), SCALE)
    with pytest.raises(VlaError, match="VLA_EINVAL"):
        S.model.lora_merge(inputs.TINY.n_layers, "wq", w0, a, b, SCALE)
    with pytest.raises(VlaError, match="VLA_EINVAL"):
        S.model.lora_merge(0, "wq", w0, a, b, float("nan"))


def test_lora_merge_7b_width_sampled_rows():
    """One decoder layer at the OpenVLA-7B width (d 4096, FFN 11008, head_dim
    128), rank 32: sampled rows of every packed projection, including the
    first and last rows of each part and of each rotary block."""
    cfg = inputs.L7B_B8.replace(name="7b_1layer", n_layers=1, batch=1)
    S = Setup(cfg, seed=3, max_batch=1)
    ad = inputs.make_lora(cfg, 32, seed=3, device="cuda")
    _merge_all(S, ad, SCALE, [0])
    adc = {k: (a.cpu(), b.cpu()) for k, (a, b) in ad[0].items()}
    rng = np.random.default_rng(3)
    for which in (5, 6, 7, 8):
        R, _ = _packed_shape(cfg, which)
        rows = sorted(set(rng.integers(0, R, 48).tolist()) | {0, 31, 32, 63, 64, R // 3, R // 3 - 1, R - 1})
        buf = _read_packed(S.model, cfg, which, 0)
        _check_packed(cfg, buf, which, rows, S.wc["layers"][0], adc, SCALE, f"7b w{which}")
    S.model.close()
