"""Passes over few rows (at most 128 suffix tokens) against the oracle where the projections' tilings change: row counts
around every 16-row block and both halvings over two workgroups, gate/up widths that take five, four and one tile per
workgroup, k ranges that are cut into slices, models wide enough for two tiles per workgroup, write-back included."""
import dataclasses

import numpy as np
import pytest
import torch

import confspec_workloads as W
from oracle import confspec_oracle as O
from paper_2602_18447_amd import binding as cb
from paper_2602_18447_amd.runner import Verifier
from tests import gpu_cases as G
from tests.test_gpu_append import _check_appended

pytestmark = pytest.mark.gpu

SHAPES = {
    "five_tiles_cut_k": dict(d_model=512, n_q_heads=4, n_kv_heads=2, d_ffn=8960),
    "four_tiles_cut_k": dict(d_model=256, n_q_heads=6, n_kv_heads=1, d_ffn=8192),
    "three_tiles_cut_k": dict(d_model=768, n_q_heads=4, n_kv_heads=2, d_ffn=8192),
    "two_tiles_cut_k": dict(d_model=2048, n_q_heads=4, n_kv_heads=2, d_ffn=8192),
    "one_tile": dict(d_model=640, n_q_heads=5, n_kv_heads=5, d_ffn=832),
    "wide": dict(d_model=4096, n_q_heads=32, n_kv_heads=4, d_ffn=1088),
}


def _parity(wl, change=None):
    """Against the oracle, on the kernels for few rows whatever the model's width."""
    weights, batch, kv = G.build_inputs(wl)
    if change:
        change(weights)
    ver = Verifier(wl.model, weights)
    cb.confspec_tune(ver.ctx, "decode_kernels", 2)
    gpu = G.run_gpu(wl, weights, batch, kv, verifier=ver)
    ver.close()
    G.compare(wl, gpu, G.run_oracle(wl, weights, batch, kv, gpu["taus"], gpu["vids"]), wl.name)


@pytest.mark.parametrize("shape", list(SHAPES))
@pytest.mark.parametrize("suffix", [(1,), (15,), (16,), (10, 7), (32,), (1,) * 33, (48, 1), (64,), (3, 62), (96,), (50, 47), (128,), (64, 65)],
                         ids=lambda s: f"T{sum(s)}")
def test_few_rows_match_oracle(shape, suffix):
    print(f"few rows: {shape}, suffixes {suffix}", flush=True)
    prefix = [(37 * i + 5) % 150 for i in range(len(suffix))]
    wl = W.tiny_workload("few_rows", 9300 + sum(suffix), dtype="bf16", n_layers=2, head_dim=128, vocab=512, block_size=16,
                         prefix_lens=prefix, suffix_lens=suffix, taus=(0.5, 0.6, 0.9), **SHAPES[shape])
    G.parity_case(wl) if wl.model.d_model <= 1792 else _parity(wl)


@pytest.mark.parametrize("suffix", [(1, 1, 1), (20, 3, 40), (5, 100)], ids=lambda s: f"T{sum(s)}")
def test_few_rows_write_back_and_repeat(suffix):
    print(f"few rows with write-back: suffixes {suffix}", flush=True)
    wl = W.tiny_workload("few_rows_append", 9400 + sum(suffix), dtype="bf16", n_layers=3, d_model=512, n_q_heads=4, n_kv_heads=2,
                         head_dim=128, d_ffn=8960, vocab=512, block_size=16, prefix_lens=[30 + 9 * i for i in range(len(suffix))],
                         suffix_lens=suffix, taus=(0.5,))
    weights = W.make_weights(wl.model, wl.seed, G.DEV)
    batch = W.make_batch(wl, G.DEV, extra_rows=max(suffix))
    kv = W.make_seeded_kv(wl, batch, G.DEV)
    before = kv.k_pages.clone(), kv.v_pages.clone()
    n_app = [min(s, 2 + 5 * i) for i, s in enumerate(suffix)]
    vids = W.draw_verdict_ids(wl)
    ver = Verifier(wl.model, weights)
    plain = [t.clone() for t in ver.verify(kv, batch, vids, [0.5])]
    outs = [t.clone() for t in ver.verify_append(kv, batch, n_app, vids, [0.5])]
    again = ver.verify_append(kv, batch, n_app, vids, [0.5])
    torch.cuda.synchronize()
    for a, b, c in zip(plain, outs, again):
        assert torch.equal(a, b) and torch.equal(b, c)
    ora = O.append_rows(wl.model, W.OracleModelView(weights), W.OracleKVView(W.KVCache(*before, wl.block_size), batch), wl.block_size,
                        batch.suffix_ids.cpu().numpy(), batch.h_cu_suffix, batch.h_prefix_lens, n_app)
    _check_appended(wl, batch, kv, before, n_app, ora, wl.name)
    ver.close()


@pytest.mark.parametrize("suffix", [(20,), (40, 9), (64, 1), (128,)], ids=lambda s: f"T{sum(s)}")
def test_few_rows_of_a_wide_model_with_few_heads(suffix):
    """A QKV projection of fewer than 128 column tiles over 128 k-tiles (d_model 8192, 12 heads).  The bound on the logits is one
    for the real models' (0.02 sqrt(1536 .. 5120), 0.8 to 1.4); at this width they are 1.8, so the head is halved."""
    print(f"few rows, wide model with few heads: suffixes {suffix}", flush=True)
    wl = W.tiny_workload("few_rows_narrow_qkv", 9350 + sum(suffix), dtype="bf16", n_layers=2, d_model=8192, n_q_heads=10, n_kv_heads=1,
                         head_dim=128, d_ffn=192, vocab=512, block_size=16, prefix_lens=[50] * len(suffix), suffix_lens=suffix,
                         taus=(0.5, 0.6, 0.9))
    _parity(wl, lambda weights: weights.lm_head.mul_(0.5))


@pytest.mark.parametrize("d_model,T,few", [(1792, 128, True), (2048, 96, True), (2048, 97, False), (2176, 64, True), (2176, 65, False), (4096, 64, True), (4096, 65, False),
                                           (4224, 32, True), (4224, 33, False)])
def test_wide_models_take_these_kernels_up_to_the_rows_where_they_win(d_model, T, few):
    """Only the general pass has RMSNorm kernels of its own (the projections for few rows carry the norms)."""
    print(f"route at width {d_model}, {T} tokens", flush=True)
    wl = W.tiny_workload("few_rows_route", 9360 + T, dtype="bf16", n_layers=2, d_model=d_model, n_q_heads=8, n_kv_heads=2, head_dim=128,
                         d_ffn=128, vocab=512, block_size=16, prefix_lens=[20], suffix_lens=[T], taus=(0.5,))
    weights, batch, kv = G.build_inputs(wl)
    ver = Verifier(wl.model, weights)
    cb.confspec_phase_timing(ver.ctx, True)
    G.run_gpu(wl, weights, batch, kv, verifier=ver)
    assert (cb.confspec_phase_times(ver.ctx)["norm"][1] == 0) == few
    ver.close()


def _one_sublayer_changes_the_rows(kind, weights):
    """A sublayer of the first layer, one with fp16 operands, moves the rows far from what they were before it."""
    m = weights.cfg
    # Where every row is c e_5 + noise, its attention output without a context is close to the value of that, v: the attention
    # can be made to add a given amount to element 5.  With a large c the same holds for the MLP and its activations.  Element 5
    # does not reach the logits itself.
    def attention_adds(c, amount):
        weights.embed[:, 5] = c
        rms = (c * c / m.d_model + 0.02 ** 2) ** 0.5
        v = weights.wqkv[0][-m.n_kv_heads * m.head_dim:, 5].float() * (c / rms) * weights.attn_norm[0][5].float()
        v = v.reshape(m.n_kv_heads, 1, m.head_dim).expand(-1, m.group, -1).reshape(-1)
        weights.wo[0][5] = (amount * v / (v @ v)).to(weights.wo[0].dtype)

    if kind == "attention_grows":
        attention_adds(0.5, 8000.0)
    elif kind == "mlp_grows":
        weights.embed[:, 5] = 8.0
        gate_up = weights.w_gate_up[0][:, 5].float() * 20.0
        act = torch.nn.functional.silu(gate_up[:m.d_ffn]) * gate_up[m.d_ffn:]
        weights.w_down[0][5] = (2.0 ** 17 * act / (act @ act)).to(weights.w_down[0].dtype)      # rms 0.4 -> 6e3
    elif kind == "attention_shrinks":
        # rms 4.2 -> 0.2 (an operand's rounding, 2^-12, leaves 96 * 2^-12 of element 5: half a percent of what is left)
        attention_adds(96.0, -96.0)
    else:                                                # from_zero_rows: padding tokens; 1 / rms is 1 / sqrt(eps)
        weights.embed.zero_()
        weights.wo[0].mul_(64.0)
    weights.final_norm[5] = 0.0


@pytest.mark.parametrize("kind", ["attention_grows", "mlp_grows", "from_zero_rows", "attention_shrinks"])
@pytest.mark.parametrize("suffix", [(1, 1, 1), (20, 9), (60, 36), (128,)], ids=lambda s: f"T{sum(s)}")
@pytest.mark.parametrize("d_ffn", [832, 8960], ids=["F832", "F8960"])
def test_rows_that_one_sublayer_grows_or_shrinks(kind, suffix, d_ffn):
    """The operand of the next projection carries a power of two of the row before the sublayer; these rows leave a half's range
    with it.  Their logits are of any size, so each trace's differences are taken over its rms on 8 verdict tokens; the bound on
    the real models' logits (rms 0.8 to 1.4) is that over 0.8."""
    print(f"few rows, {kind}: suffixes {suffix}, d_ffn {d_ffn}", flush=True)
    prefix = [37 * i + 5 if kind == "from_zero_rows" else 0 for i in range(len(suffix))]
    wl = W.tiny_workload("few_rows_" + kind, 9450 + sum(suffix), dtype="bf16", n_layers=4, d_model=512, n_q_heads=4, n_kv_heads=2,
                         head_dim=128, d_ffn=d_ffn, vocab=512, block_size=16, prefix_lens=prefix, suffix_lens=suffix, n_verdict=8)
    if kind == "from_zero_rows":
        wl = dataclasses.replace(wl, model=dataclasses.replace(wl.model, rms_eps=1e-12))
    weights, batch, kv = G.build_inputs(wl)
    _one_sublayer_changes_the_rows(kind, weights)
    gpu = G.run_gpu(wl, weights, batch, kv)
    ora = G.run_oracle(wl, weights, batch, kv, gpu["taus"], gpu["vids"])
    worst = float((np.abs(gpu["logits"] - ora["logits"]) / np.sqrt((ora["logits"] ** 2).mean(axis=1, keepdims=True))).max())
    print(f"{wl.name}: largest logit difference {worst:.4f}", flush=True)
    assert worst <= G.TOL["bf16"]["logit"] / 0.8
