"""fp32 path: whole pass against the oracle where its tiles can go wrong - row counts around 16 and 32, query rows of
several q heads per kv head, both head sizes, page sizes that do not divide a tile, and widths that take the 32 x 32 tiles."""
import pytest
import torch

import confspec_workloads as W
from paper_2602_18447_amd.runner import Verifier
from tests import gpu_cases as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("heads,hd,block,prefix,suffix", [
    ((4, 4), 64, 16, (0, 1, 127), (1, 15, 16)),
    ((6, 2), 64, 7, (33, 0), (17, 33)),
    ((4, 1), 128, 16, (16, 5, 300), (1, 31, 40)),
    ((6, 3), 128, 5, (64,), (130,)),
    ((4, 4), 64, 32, (200, 31), (20, 63)),                                       # 192 keys of a round and past them; a block of two tiles
    ((4, 4), 64, 48, (47, 0, 90, 16, 33, 1, 49, 96), (130, 20, 64, 5, 97, 33, 80, 70)),      # a grid of more workgroups than CUs, 32 x 32 tiles of narrow outputs
    ((6, 2), 128, 32, (70, 33), (33, 8)),
    ((4, 4), 64, 7, (47, 0, 90, 16, 33, 1, 49, 300), (130, 20, 64, 5, 97, 33, 80, 70)),      # such a grid, blocks that do not divide a tile
])
@pytest.mark.parametrize("d_ffn", [96, 4096])
def test_fp32_pass_matches_oracle(heads, hd, block, prefix, suffix, d_ffn):
    print(f"fp32 pass heads={heads} hd={hd} block={block} L={prefix} S={suffix} F={d_ffn}", flush=True)
    wl = W.tiny_workload("f32_tiles", 9100 + hd + d_ffn, dtype="fp32", n_layers=2, d_model=320, n_q_heads=heads[0], n_kv_heads=heads[1],
                         head_dim=hd, d_ffn=d_ffn, vocab=512, block_size=block, prefix_lens=prefix, suffix_lens=suffix,
                         taus=(0.5, 0.6, 0.9))
    G.parity_case(wl)


@pytest.mark.parametrize("hd", [64, 128])
@pytest.mark.parametrize("value", [float("nan"), float("inf")], ids=str)
def test_fp32_later_tokens_do_not_reach_earlier_ones(hd, value):
    """A suffix token with a NaN or an infinity in its embedding row: the keys and values of the tokens before it, in its own and
    in the other traces, are the bits that they are without it."""
    print(f"fp32 pass with {value} in a later token, head size {hd}", flush=True)
    suffix, bad = (20, 33, 5), 20 + 25
    wl = W.tiny_workload("f32_mask", 9150 + hd, dtype="fp32", n_layers=3, d_model=320, n_q_heads=6, n_kv_heads=2, head_dim=hd, d_ffn=96,
                         vocab=512, block_size=16, prefix_lens=(33, 5, 0), suffix_lens=suffix, taus=(0.5,))
    weights = W.make_weights(wl.model, wl.seed, G.DEV)
    batch = W.make_batch(wl, G.DEV, extra_rows=max(suffix))
    batch.suffix_ids[batch.suffix_ids == 511] = 510
    batch.suffix_ids[bad] = 511
    pages = []
    for v in (0.25, value):
        weights.embed[511].fill_(0.25)
        weights.embed[511, 7] = v
        kv = W.make_seeded_kv(wl, batch, G.DEV)
        ver = Verifier(wl.model, weights)
        ver.verify_append(kv, batch, list(suffix), W.draw_verdict_ids(wl), [0.5])
        torch.cuda.synchronize()
        pages.append((kv.k_pages.clone(), kv.v_pages.clone()))
        ver.close()
    table = batch.block_table.cpu().numpy()
    for b, (L, S) in enumerate(zip(wl.prefix_lens, suffix)):
        for i in range(S):
            row = L + i
            at = (slice(None), int(table[b, row // 16]), slice(None), row % 16)
            for clean, odd in zip(*pages):
                if b != 1 or i < bad - 20:
                    assert torch.equal(clean[at], odd[at]), (b, i)
                else:
                    assert not torch.isfinite(odd[at][1:]).all(), (b, i)
