"""Passes over few rows (at most 128 suffix tokens) against the oracle where the projections' tilings change: row counts
around every 16-row block and both halvings over two workgroups, gate/up widths that take five, four and one tile per
workgroup, k ranges that are cut into slices, models wide enough for two tiles per workgroup, write-back included."""
import pytest
import torch

import confspec_workloads as W
from oracle import confspec_oracle as O
from paper_2602_18447_amd.runner import Verifier
from tests import gpu_cases as G
from tests.test_gpu_append import _check_appended

pytestmark = pytest.mark.gpu

SHAPES = {
    "five_tiles_cut_k": dict(d_model=512, n_q_heads=4, n_kv_heads=2, d_ffn=8960),
    "four_tiles_cut_k": dict(d_model=256, n_q_heads=6, n_kv_heads=1, d_ffn=8192),
    "one_tile": dict(d_model=640, n_q_heads=5, n_kv_heads=5, d_ffn=832),
    "wide": dict(d_model=4096, n_q_heads=32, n_kv_heads=4, d_ffn=1088),
}


@pytest.mark.parametrize("shape", list(SHAPES))
@pytest.mark.parametrize("suffix", [(1,), (15,), (16,), (10, 7), (32,), (1,) * 33, (48, 1), (64,), (3, 62), (96,), (50, 47), (128,), (64, 65)],
                         ids=lambda s: f"T{sum(s)}")
def test_few_rows_match_oracle(shape, suffix):
    print(f"few rows: {shape}, suffixes {suffix}", flush=True)
    prefix = [(37 * i + 5) % 150 for i in range(len(suffix))]
    wl = W.tiny_workload("few_rows", 9300 + sum(suffix), dtype="bf16", n_layers=2, head_dim=128, vocab=512, block_size=16,
                         prefix_lens=prefix, suffix_lens=suffix, taus=(0.5, 0.6, 0.9), **SHAPES[shape])
    G.parity_case(wl)


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
    """A QKV projection of fewer than 128 column tiles over 128 k-tiles (d_model 8192, 12 heads)."""
    print(f"few rows, wide model with few heads: suffixes {suffix}", flush=True)
    wl = W.tiny_workload("few_rows_narrow_qkv", 9350 + sum(suffix), dtype="bf16", n_layers=2, d_model=8192, n_q_heads=10, n_kv_heads=1,
                         head_dim=128, d_ffn=192, vocab=512, block_size=16, prefix_lens=[50] * len(suffix), suffix_lens=suffix,
                         taus=(0.5, 0.6, 0.9))
    G.parity_case(wl)
