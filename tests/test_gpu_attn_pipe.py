"""The pipelined attention loop where its exponent reference has to move: rows whose running maximum starts far below zero, rises by
hundreds chunk by chunk, or stays low, whole items and pieces; one key with most of the weight, and values of extreme size; against the
oracle."""
import numpy as np
import pytest
import torch

import confspec_workloads as W
from oracle import confspec_oracle as O
from paper_2602_18447_amd import binding as cb
from tests.test_gpu_ops import _batch_structs, _ctx, _rand, f64

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

# score of a key (log2 units, before noise of a few units) by 64-key chunk, for a query along +1; queries go along +1, -1 and 0.3
PROFILES = {
    "rising": (-400, -300, -190, -120, -60, 0, 30, 63, 66, 129, 300),
    "falling": (300, 129, 66, 0, -70, -150, -400),
    "low": (-70, -80, -65, -300),
    "flat": (0, 3, -2, 1),
    "edge": (64, 64, 65, -64, -65, 128, 129),
}


@pytest.mark.parametrize("split", [1, 3])
@pytest.mark.parametrize("name", sorted(PROFILES))
def test_scores_past_the_reference_range(name, split):
    print(f"attention reference range {name} split={split}", flush=True)
    prof = PROFILES[name]
    L, hq, hkv, hd, S = 64 * len(prof) - 5, 12, 2, 128, (40, 1, 130)
    wl = W.tiny_workload("range", 91, dtype="bf16", n_layers=1, n_q_heads=hq, n_kv_heads=hkv, head_dim=hd, d_model=256,
                         prefix_lens=(L, L, L), suffix_lens=S, block_size=16)
    ctx, _ = _ctx("bf16", n_layers=1, n_q_heads=hq, n_kv_heads=hkv, head_dim=hd)
    cb.confspec_tune(ctx, "attn_kernel", 2)
    cb.confspec_tune(ctx, "attn_min_chunks", 1)
    cb.confspec_tune(ctx, "attn_split", split)
    batch, T = W.make_batch(wl, DEV), wl.T
    kv = W.make_seeded_kv(wl, batch, DEV)
    u = torch.zeros(hd, device=DEV)
    u[::2] = 1.0                                                      # 64 elements
    per_unit = 64 * 8.0 / np.sqrt(hd) * np.log2(np.e)                 # score of a key u / 8 .. for a query 8 u
    for b in range(wl.B):
        for p in range((L + 15) // 16):
            kv.k_pages[0, int(batch.block_table[b, p])] += (prof[min(p // 4, len(prof) - 1)] / per_unit * u).to(torch.bfloat16)
    along = torch.tensor([8.0, -8.0, 2.4], device=DEV)[torch.arange(hq, device=DEV) % 3]
    q = (_rand((T, hq, hd), torch.float32, 92, 0.3) + along[None, :, None] * u).to(torch.bfloat16)
    ks = (_rand((T, hkv, hd), torch.float32, 93, 0.5) + prof[-1] / per_unit * u).to(torch.bfloat16)
    vs = _rand((T, hkv, hd), torch.bfloat16, 94, 0.5)
    out = torch.zeros((T, hq * hd), dtype=torch.bfloat16, device=DEV)
    kvs = cb.make_kv(kv.k_pages, kv.v_pages, batch.block_table, batch.n_blocks, 16, batch.max_blocks_per_seq)
    bs, keep = _batch_structs(wl, batch)
    ws = torch.empty(cb.confspec_workspace_bytes(ctx, T, wl.B), dtype=torch.uint8, device=DEV)
    cb.confspec_op_attention(ctx, kvs, bs, 0, q, ks, vs, out, ws)
    torch.cuda.synchronize()
    view, got = W.OracleKVView(kv, batch), f64(out).reshape(T, hq, hd)
    for b in range(wl.B):
        ids = batch.block_table[b, :(L + 15) // 16].cpu().numpy()
        t0, t1 = int(batch.h_cu_suffix[b]), int(batch.h_cu_suffix[b + 1])
        k_all = np.concatenate([O.gather_prefix(view.k_blocks(0, ids), L), f64(ks)[t0:t1]])
        v_all = np.concatenate([O.gather_prefix(view.v_blocks(0, ids), L), f64(vs)[t0:t1]])
        ref = O.attention(f64(q)[t0:t1], k_all, v_all, L)
        # probabilities and the result rounded to 8 mantissa bits; fp32 scores of some hundred: 2^-15 relative in a probability
        assert np.abs(got[t0:t1] - ref).max() <= (3 * 2.0 ** -9 + 2.0 ** -13) * np.abs(v_all).max(), (name, b)
    cb.confspec_destroy(ctx)


# suffixes of one to nine chunks, whole items and pieces that begin inside the suffix, chunk boundaries on either side
@pytest.mark.parametrize("split", [1, 4])
@pytest.mark.parametrize("prefix_lens,suffix_lens", [((40, 0, 700), (300, 65, 128)), ((64, 129), (513, 64))])
def test_second_terms_of_several_suffix_chunks(prefix_lens, suffix_lens, split, monkeypatch):
    print(f"two-term attention L={prefix_lens} S={suffix_lens} split={split}", flush=True)
    from tests import test_gpu_ops

    def ctx_with_split(*args, **kw):
        ctx, cfg = _ctx(*args, **kw)
        cb.confspec_tune(ctx, "attn_min_chunks", 1)
        cb.confspec_tune(ctx, "attn_split", split)
        return ctx, cfg

    monkeypatch.setattr(test_gpu_ops, "_ctx", ctx_with_split)
    # as for short suffixes: two terms are 16 bits of mantissa, 2^-17 relative in q and k, scores of up to about 20
    assert test_gpu_ops._attention_case("bf16", 12, 2, 128, prefix_lens, suffix_lens, out_terms=2, precise=True) <= 2e-4


# partial results with room for 32, 64, 96 and 128 rows (the largest tile's), pieces without chunks among them
@pytest.mark.parametrize("kernel", [1, 2])
@pytest.mark.parametrize("suffix_lens", [(1, 5, 2, 1), (1, 9, 2, 10), (3, 1, 16, 11), (17, 1, 21, 2), (1, 22, 64, 3)])
def test_partial_results_of_few_rows(suffix_lens, kernel, monkeypatch):
    print(f"attention partial results S={suffix_lens} kernel={kernel}", flush=True)
    from tests import test_gpu_ops

    def ctx_with_split(*args, **kw):
        ctx, cfg = _ctx(*args, **kw)
        for key, val in (("attn_kernel", kernel), ("attn_min_chunks", 1), ("attn_split", 4)):
            cb.confspec_tune(ctx, key, val)
        return ctx, cfg

    monkeypatch.setattr(test_gpu_ops, "_ctx", ctx_with_split)
    # as for other suffixes (tests/test_gpu_ops.py)
    assert test_gpu_ops._attention_case("bf16", 12, 2, 128, (1700, 64, 900, 0), suffix_lens) <= 6e-3
    assert test_gpu_ops._attention_case("bf16", 12, 2, 128, (1700, 64, 900, 0), suffix_lens, out_terms=2, precise=True) <= 2e-4


def _attend(L, S, seed, split, offset_of_key, spread, value, along, out_terms=1, kernel=2, two_term=False):
    """Attention of suffixes S behind contexts of L keys (a key: offset_of_key(i) score units along u, plus noise; a value: value(noise, key));
    row r of head h of q goes along[(r + h) % len(along)] of u.  Returns the result and the oracle's, [T, Hq, 128]."""
    hq, hkv, hd = 12, 2, 128
    lo = {n: torch.zeros((sum(S), h, hd), dtype=torch.bfloat16, device=DEV) for n, h in (("q_lo", hq), ("k_lo", hkv), ("v_lo", hkv))}
    wl = W.tiny_workload("range", seed, dtype="bf16", n_layers=1, n_q_heads=hq, n_kv_heads=hkv, head_dim=hd, d_model=256,
                         prefix_lens=(L,) * len(S), suffix_lens=S, block_size=16)
    ctx, _ = _ctx("bf16", n_layers=1, n_q_heads=hq, n_kv_heads=hkv, head_dim=hd)
    cb.confspec_tune(ctx, "attn_kernel", kernel)
    cb.confspec_tune(ctx, "attn_min_chunks", 1)
    cb.confspec_tune(ctx, "attn_split", split)
    batch, T = W.make_batch(wl, DEV), wl.T
    kv = W.make_seeded_kv(wl, batch, DEV)                             # N(0, 0.5): scaled below
    u = torch.zeros(hd, device=DEV)
    u[::2] = 1.0                                                      # 64 elements
    per_unit = 64 * 8.0 / np.sqrt(hd) * np.log2(np.e)                 # score (log2 units) of a key u / 8 .. for a query 8 u
    keys = torch.arange(batch.max_blocks_per_seq * 16, device=DEV)
    off, vcol = offset_of_key(keys).float() / per_unit, keys.view(-1, 16)
    for b in range(wl.B):
        for p in range((L + 15) // 16):
            blk = int(batch.block_table[b, p])
            k, v = kv.k_pages[0, blk].float(), kv.v_pages[0, blk].float()
            kv.k_pages[0, blk] = (2 * spread * k + off[16 * p:16 * p + 16, None] * u).to(torch.bfloat16)
            kv.v_pages[0, blk] = value(2 * v, vcol[p][:, None]).to(torch.bfloat16)
    a = torch.tensor(along, device=DEV)[(torch.arange(T, device=DEV)[:, None] + torch.arange(hq, device=DEV)) % len(along)]
    q = (_rand((T, hq, hd), torch.float32, seed + 1, 0.3) + 8.0 * a[..., None] * u).to(torch.bfloat16)
    later = torch.full((1, 1, 1), L, device=DEV)
    ks = (_rand((T, hkv, hd), torch.float32, seed + 2, spread) + float(offset_of_key(later)) / per_unit * u).to(torch.bfloat16)
    vs = value(_rand((T, hkv, hd), torch.float32, seed + 3), later).to(torch.bfloat16)
    out = torch.zeros((T, out_terms * hq * hd), dtype=torch.bfloat16, device=DEV)
    kvs = cb.make_kv(kv.k_pages, kv.v_pages, batch.block_table, batch.n_blocks, 16, batch.max_blocks_per_seq)
    bs, keep = _batch_structs(wl, batch)
    ws = torch.empty(cb.confspec_workspace_bytes(ctx, T, wl.B), dtype=torch.uint8, device=DEV)
    cb.confspec_op_attention(ctx, kvs, bs, 0, q, ks, vs, out, ws, out_terms=out_terms, **(lo if two_term else {}))
    torch.cuda.synchronize()
    got = f64(out).reshape(T, out_terms, hq, hd).sum(axis=1)
    view, ref = W.OracleKVView(kv, batch), np.zeros((T, hq, hd))
    for b in range(wl.B):
        ids = batch.block_table[b, :(L + 15) // 16].cpu().numpy()
        t0, t1 = int(batch.h_cu_suffix[b]), int(batch.h_cu_suffix[b + 1])
        k_all = np.concatenate([O.gather_prefix(view.k_blocks(0, ids), L), f64(ks)[t0:t1]])
        v_all = np.concatenate([O.gather_prefix(view.v_blocks(0, ids), L), f64(vs)[t0:t1]])
        ref[t0:t1] = O.attention(f64(q)[t0:t1], k_all, v_all, L)
    cb.confspec_destroy(ctx)
    return got, ref


@pytest.mark.parametrize("split", [1, 3])
def test_a_key_with_most_of_the_weight_and_no_value(split):
    """The first key takes about half to nine tenths of every row's weight and has no value, the other 1100 have values about 1.  The result is
    the others' share: rounding of the first key's probability in the normaliser, or off the reference, would show in full."""
    print(f"attention sink split={split}", flush=True)
    L, S = 1100, (70, 33)
    along = [1.0 + 0.01 * i for i in range(-9, 10)]                   # the first key's score differs from row to row
    got, ref = _attend(L, S, 95, split, lambda i: 11.0 * (i == 0), 0.12, lambda x, i: (1.0 + 0.25 * x) * (i > 0), along, out_terms=2)
    assert 0.02 < ref.min() and ref.max() < 0.9                       # q's own noise moves the share, too
    # the others' probabilities are rounded to 8 mantissa bits: 2^-9 / sqrt(3) relative each, independent, spread over about a factor of
    # two (rms to mean 1.3) - six standard deviations of the mean of 1100; fp32 sums of 1100 terms and the two-term result 2^-15
    bound = 6 * 2.0 ** -9 / np.sqrt(3.0) * 1.3 / np.sqrt(L) + 2.0 ** -15
    assert (np.abs(got - ref) / ref).max() <= bound


@pytest.mark.parametrize("split", [1, 3])
@pytest.mark.parametrize("size", [2.0 ** 100, 2.0 ** -110])
def test_values_of_extreme_size(size, split):
    """Rows whose scores all lie near +50, or near -50 (log2 units): neither large nor small values leave the range."""
    print(f"attention values {size:g} split={split}", flush=True)
    got, ref = _attend(1000, (40, 1, 130), 97, split, lambda i: 50.0 + 0 * i, 0.12, lambda x, i: size * x, [1.0, -1.0])
    assert np.abs(got - ref).max() <= (3 * 2.0 ** -9 + 2.0 ** -13) * np.abs(ref).max()


@pytest.mark.parametrize("split", [1, 3])
@pytest.mark.parametrize("kernel,two_term", [(1, False), (2, False), (0, True)])
def test_first_keys_far_below_zero(kernel, two_term, split):
    """Every loop: the first 64 keys score about -400 for half of the rows, so exp2 of minus their maximum is not a number to scale by."""
    print(f"attention low first keys kernel={kernel} two_term={two_term} split={split}", flush=True)
    got, ref = _attend(700, (40, 1, 130), 99, split, lambda i: -400.0 * (i < 64), 0.12, lambda x, i: x, [1.0, -1.0], kernel=kernel, two_term=two_term)
    # as above; the +400 of the other rows makes fp32 scores of some hundred: 2^-15 relative in a probability
    assert np.abs(got - ref).max() <= (3 * 2.0 ** -9 + 2.0 ** -13) * np.abs(ref).max()
