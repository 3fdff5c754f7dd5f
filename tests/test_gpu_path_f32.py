"""fp32 path: whole pass against the oracle where its tiles can go wrong - row counts around 16 and 32, query rows of
several q heads per kv head, both head sizes, page sizes that do not divide a tile, and widths that take the 32 x 32 tiles."""
import pytest

import confspec_workloads as W
from tests import gpu_cases as G

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("heads,hd,block,prefix,suffix", [
    ((4, 4), 64, 16, (0, 1, 127), (1, 15, 16)),
    ((6, 2), 64, 7, (33, 0), (17, 33)),
    ((4, 1), 128, 16, (16, 5, 300), (1, 31, 40)),
    ((6, 3), 128, 5, (64,), (130,)),
])
@pytest.mark.parametrize("d_ffn", [96, 4096])
def test_fp32_pass_matches_oracle(heads, hd, block, prefix, suffix, d_ffn):
    print(f"fp32 pass heads={heads} hd={hd} block={block} L={prefix} S={suffix} F={d_ffn}", flush=True)
    wl = W.tiny_workload("f32_tiles", 9100 + hd + d_ffn, dtype="fp32", n_layers=2, d_model=320, n_q_heads=heads[0], n_kv_heads=heads[1],
                         head_dim=hd, d_ffn=d_ffn, vocab=512, block_size=block, prefix_lens=prefix, suffix_lens=suffix,
                         taus=(0.5, 0.6, 0.9))
    G.parity_case(wl)
