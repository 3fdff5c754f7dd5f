"""Attention of passes over at most 128 suffix tokens against the oracle where its cut of rows and keys changes: contexts
around page, round and piece borders, tiles that end inside a token's heads, suffixes around the 32-row and 16-key
borders, one piece for context and suffix together (many tiles), groups of candidates on one context."""
import numpy as np
import pytest
import torch

import confspec_workloads as W
from paper_2602_18447_amd import binding as cb
from paper_2602_18447_amd.runner import Verifier
from tests import gpu_cases as G
from tests.test_gpu_verify import _shared_case

pytestmark = pytest.mark.gpu

HEADS = {"G1": (4, 4), "G5": (5, 1), "G6": (12, 2), "G16": (16, 1)}


def _wl(name, seed, heads, prefix, suffix):
    hq, hkv = HEADS[heads]
    return W.tiny_workload(name, seed, dtype="bf16", n_layers=3, d_model=512, n_q_heads=hq, n_kv_heads=hkv, head_dim=128, d_ffn=768,
                           vocab=512, block_size=16, prefix_lens=prefix, suffix_lens=suffix, taus=(0.5, 0.55, 0.6, 0.9))


@pytest.mark.parametrize("heads", list(HEADS))
@pytest.mark.parametrize("batch", [
    ((0,), (5,)), ((1, 0), (2, 33)), ((15, 16, 17, 255), (6, 7, 11, 17)), ((256, 257, 511, 512, 513), (16, 17, 31, 32, 32)),
    ((4097,), (96,)), ((700, 31), (1, 127)), ((300,) * 40, (3,) * 40), ((5, 2040, 90), (1, 1, 1)), ((640,) * 64, (2,) * 64),
], ids=lambda b: f"B{len(b[0])}T{sum(b[1])}L{max(b[0])}")
def test_few_row_attention_matches_oracle(heads, batch):
    print(f"few-row attention: {heads}, prefixes {batch[0]}, suffixes {batch[1]}", flush=True)
    G.parity_case(_wl("attn_few", 9500 + sum(batch[1]), heads, *batch))


@pytest.mark.parametrize("heads", ["G1", "G6"])
def test_few_row_attention_on_shared_contexts(heads):
    print(f"few-row attention on shared contexts, {heads}", flush=True)
    hq, hkv = HEADS[heads]
    groups = [(300, (5, 1, 17)), (0, (3, 4)), (77, (9,)), (1030, (20, 33, 2, 7))]
    wl, weights, batch, kv, gstart = _shared_case("attn_few_shared", 9600, groups, n_q_heads=hq, n_kv_heads=hkv)
    taus, vids = G.sweep_taus(wl), W.draw_verdict_ids(wl)
    ver = Verifier(wl.model, weights)
    outs = ver.verify_shared(kv, batch, gstart, vids, taus)
    torch.cuda.synchronize()
    gpu = dict(logits=outs[0].cpu().numpy().astype(np.float64), conf=outs[1].cpu().numpy().astype(np.float64),
               verdict=outs[2].cpu().numpy(), accept=outs[3].cpu().numpy(), taus=taus, vids=vids)
    G.compare(wl, gpu, G.run_oracle(wl, weights, batch, kv, taus, vids), wl.name)
    ver.close()


@pytest.mark.parametrize("hq,suffix", [(64, (3, 20)), (65, (3, 20)), (96, (1, 1, 1)), (96, (33,)), (128, (1, 127))], ids=str)
def test_many_q_heads_per_kv_head(hq, suffix):
    """Around and above the q heads per kv head that the few-row attention takes (64): above, the general kernels."""
    print(f"{hq} q heads on one kv head, suffixes {suffix}", flush=True)
    wl = W.tiny_workload("attn_few_heads", 9700 + hq + sum(suffix), dtype="bf16", n_layers=3, d_model=512, n_q_heads=hq, n_kv_heads=1,
                         head_dim=128, d_ffn=768, vocab=512, block_size=16, prefix_lens=[70 + 300 * i for i in range(len(suffix))],
                         suffix_lens=suffix, taus=(0.5, 0.55, 0.6, 0.9))
    G.parity_case(wl)


# pieces of 256 keys each, which the last workgroup of a tile adds up 12 at a time, or 4 where that is all: one of them, every border of a
# round, rows taken by all threads (16 heads) or by half of them for the even and the odd pieces (up to 8 heads)
@pytest.mark.parametrize("heads", ["G5", "G6", "G16"])
@pytest.mark.parametrize("prefix", [(256,), (260,), (4 * 256, 4 * 256 + 1), (8 * 256, 8 * 256 + 1), (12 * 256,), (12 * 256 + 1, 9), (24 * 256, 24 * 256 + 3), (25 * 256 - 15,)], ids=lambda p: f"L{max(p)}")
def test_pieces_of_one_token(heads, prefix):
    print(f"pieces of one token: {heads}, prefixes {prefix}", flush=True)
    G.parity_case(_wl("attn_few_pieces", 9800 + len(prefix), heads, prefix, (1,) * len(prefix)))


# the same with five tokens, 30 rows: rounds of 8 and a rest of 2, 4, 6 or 8, the suffix's piece the last
@pytest.mark.parametrize("pieces", [1, 2, 3, 4, 5, 6, 7, 8, 9, 15, 16, 17])
def test_pieces_of_several_tokens(pieces):
    print(f"pieces of five tokens: {pieces} of the context", flush=True)
    G.parity_case(_wl("attn_few_pieces", 9850 + pieces, "G6", (256 * pieces - 3,), (5,)))


@pytest.mark.parametrize("pieces", [2, 3, 13])
@pytest.mark.parametrize("hq", [12, 32])
def test_an_infinite_value_in_the_last_piece(hq, pieces):
    """A round that is larger than what is left of the pieces reads the last one again and takes nothing of it, also where it holds an infinity.
    The layer's result is IEEE half, which an infinity leaves at the largest number: the logits stay numbers, those of the general kernels."""
    print(f"infinite value, {pieces} pieces, {hq} heads", flush=True)
    wl = W.tiny_workload("attn_few_inf", 9900 + pieces, dtype="bf16", n_layers=4, d_model=1664, n_q_heads=hq, n_kv_heads=2, head_dim=128, d_ffn=768,
                         vocab=512, block_size=16, prefix_lens=(256 * pieces - 5,), suffix_lens=(1,), taus=(0.5,))
    ver = Verifier(wl.model, W.make_weights(wl.model, wl.seed, G.DEV))
    batch, vids = W.make_batch(wl, G.DEV), W.draw_verdict_ids(wl)
    kv = W.make_seeded_kv(wl, batch, G.DEV)
    kv.v_pages[1, int(batch.block_table[0, 16 * pieces - 1]), :, 3, 17] = float("inf")        # layer 1: one-term probabilities
    logits = {}
    for kernels in (1, 0):
        cb.confspec_tune(ver.ctx, "decode_kernels", kernels)
        logits[kernels] = ver.verify(kv, batch, vids, [0.5])[0].cpu().numpy().astype(np.float64)
    print("  logits", logits, flush=True)
    assert np.isfinite(logits[0]).all()
    assert np.abs(logits[1] - logits[0]).max() <= 2.0 ** -8            # (activations of 8 bits; logits of about 1)
    ver.close()
