"""GEMMs of one round of tiles with loading wavefronts of their own: every epilogue and operand format at the edges of the
tiles, k ranges shorter than the ring of stages, uneven k slices on every tile, against the fp64 product; the reduction of the slices with
the next norm."""
import numpy as np
import pytest
import torch

import confspec_workloads as W
from oracle import confspec_oracle as O
from paper_2602_18447_amd import binding as cb
from paper_2602_18447_amd.runner import Verifier
from tests.test_gpu_ops import _ctx, _rand, f64

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _operands(M, N, K, fmt):
    full = _rand((M, K), torch.float32, 7 * M + K)
    Wt = _rand((N, K), torch.float32, 11 * N + K, 0.05).to(torch.float16 if fmt == 3 else torch.bfloat16)
    if fmt == 2:
        hi = full.to(torch.bfloat16)
        lo = (full - hi.float()).to(torch.bfloat16)
        return torch.cat([hi, lo], dim=1).contiguous(), f64(hi) + f64(lo), Wt
    A = full.to(torch.float16 if fmt == 3 else torch.bfloat16)
    return A, f64(A), Wt


# Tiles taken without slices (the host check holds the plans of every shape in this file): 64 x 64 (and 64 x 128 for SwiGLU) for the first
# five, 128 x 128 (1290 to 2040 rows), 256 x 128 (2600 x 2048, 200 x 17920), 64 x 128 (257 x 4096), 256 x 192 (7937 x 1536); rows at and
# next to the tiles' edges, one and two k-tiles (fewer than the stages), and enough of them that the ring wraps
@pytest.mark.parametrize("fmt", [1, 2, 3])
@pytest.mark.parametrize("M,N,K", [(33, 128, 64), (64, 256, 128), (65, 384, 192), (129, 512, 832), (255, 2048, 320), (1290, 2048, 128),
                                   (2040, 2048, 448), (1921, 2048, 192), (2600, 2048, 576), (257, 4096, 1024), (200, 17920, 448), (7937, 1536, 576),
                                   (10753, 1536, 192), (18606, 1536, 320),               # 256 x 256 tiles, and the rows behind them on smaller ones
                                   (1, 128, 64), (8, 33024, 320), (32, 32768, 192)])     # the last three: tiles of 32 rows
def test_one_round_tiles(M, N, K, fmt):
    print(f"feed M={M} N={N} K={K} fmt={fmt}", flush=True)
    ctx, _ = _ctx("bf16")
    A, a64, Wt = _operands(M, N, K, fmt)
    ref = a64 @ f64(Wt).T
    scale = max(np.abs(ref).max(), 4.0)
    x0 = _rand((M + 2, N), torch.float32, 5)                              # two guard rows
    nbytes = cb.confspec_op_gemm_scratch_bytes(ctx, M, N, K, fmt)
    for scratch in [None] + ([torch.empty(nbytes, dtype=torch.uint8, device=DEV)] if nbytes else []):
        x, st = x0.clone(), torch.full_like(x0, 7.0)
        cb.confspec_op_gemm(ctx, A, Wt, x, M, N, K, cb.EPI_RESID_F32, fmt, 1, scratch)
        cb.confspec_op_gemm(ctx, A, Wt, st, M, N, K, cb.EPI_STORE_F32, fmt, 1, scratch)
        F = N // 2
        act = torch.zeros((M + 1, (2 if fmt == 2 else 1) * F), dtype=torch.float16 if fmt == 3 else torch.bfloat16, device=DEV)
        cb.confspec_op_gemm(ctx, A, Wt, act, M, N, K, cb.EPI_SWIGLU, fmt, fmt, scratch)
        torch.cuda.synchronize()
        assert np.abs(f64(x[:M]) - ref - f64(x0[:M])).max() <= 2e-5 * scale and torch.equal(x[M:], x0[M:])
        assert np.abs(f64(st[:M]) - ref).max() <= 2e-5 * scale and torch.all(st[M:] == 7.0)
        r3 = ref.reshape(M, N // 64, 2, 32)
        want = (O.silu(r3[:, :, 0, :]) * r3[:, :, 1, :]).reshape(M, F)
        got = f64(act[:M, :F]) + (f64(act[:M, F:]) if fmt == 2 else 0.0)
        # one rounding to 8 (11, 16) mantissa bits, and the fp32 product's error through the activation
        assert np.all(np.abs(got - want) <= 2.0 ** {1: -8, 2: -15, 3: -11}[fmt] * np.abs(want) + 1e-4 * np.abs(want).max())
        assert torch.all(act[M:] == 0)
    cb.confspec_destroy(ctx)


# k slices that do not divide the k-tiles, one shape for each tile: 64 x 64 (6 slices), 64 x 128 (5), 128 x 128 (8), 256 x 128 (3), 256 x 192 (4)
SLICED = [(33, 256, 1664), (65, 3072, 2432), (66, 3072, 2944), (641, 3072, 2816), (769, 3072, 4224)]


@pytest.mark.parametrize("fmt", [1, 2, 3])
@pytest.mark.parametrize("M,N,k_total", SLICED)
def test_sliced_tiles(M, N, k_total, fmt):
    K = k_total // (2 if fmt == 2 else 1)                                 # two terms: every k-tile of W meets two of A
    print(f"feed sliced M={M} N={N} K={K} fmt={fmt}", flush=True)
    ctx, _ = _ctx("bf16")
    A, a64, Wt = _operands(M, N, K, fmt)
    ref = a64 @ f64(Wt).T
    scale = max(np.abs(ref).max(), 4.0)
    x0 = _rand((M + 2, N), torch.float32, 5)                              # two guard rows
    nbytes = cb.confspec_op_gemm_scratch_bytes(ctx, M, N, K, fmt)
    assert nbytes > 2 * M * N * 4                                         # three slices and more
    scratch = torch.full((nbytes + 256,), 0xff, dtype=torch.uint8, device=DEV)   # NaN where a slice would not be written
    F = N // 2
    runs = []
    for group_m in (0, 1, 3):                                             # the tile order is not the sums' order
        cb.confspec_tune(ctx, "gemm_group_m", group_m)
        scratch[:nbytes].fill_(0xff)
        x, st = x0.clone(), torch.full_like(x0, 7.0)
        act = torch.zeros((M + 1, (2 if fmt == 2 else 1) * F), dtype=torch.float16 if fmt == 3 else torch.bfloat16, device=DEV)
        cb.confspec_op_gemm(ctx, A, Wt, x, M, N, K, cb.EPI_RESID_F32, fmt, 1, scratch[:nbytes])
        cb.confspec_op_gemm(ctx, A, Wt, st, M, N, K, cb.EPI_STORE_F32, fmt, 1, scratch[:nbytes])
        cb.confspec_op_gemm(ctx, A, Wt, act, M, N, K, cb.EPI_SWIGLU, fmt, fmt, scratch[:nbytes])
        torch.cuda.synchronize()
        assert torch.all(scratch[nbytes:] == 0xff)
        runs.append((x, st, act))
    for other in runs[1:]:
        assert all(torch.equal(a, b) for a, b in zip(runs[0], other))
    x, st, act = runs[0]
    assert np.abs(f64(x[:M]) - ref - f64(x0[:M])).max() <= 2e-5 * scale and torch.equal(x[M:], x0[M:])
    assert np.abs(f64(st[:M]) - ref).max() <= 2e-5 * scale and torch.all(st[M:] == 7.0)
    r3 = ref.reshape(M, N // 64, 2, 32)
    want = (O.silu(r3[:, :, 0, :]) * r3[:, :, 1, :]).reshape(M, F)
    got = f64(act[:M, :F]) + (f64(act[:M, F:]) if fmt == 2 else 0.0)
    # as above
    assert np.all(np.abs(got - want) <= 2.0 ** {1: -8, 2: -15, 3: -11}[fmt] * np.abs(want) + 1e-4 * np.abs(want).max())
    assert torch.all(act[M:] == 0)
    cb.confspec_destroy(ctx)


@pytest.mark.parametrize("fmt", [1, 2, 3])
@pytest.mark.parametrize("lens", [(40, 33, 1), (130, 127), (1500, 541), (2600,)])   # 64 x 64 tiles (74 and 257 rows), 128 x 128, 256 x 128
def test_rotating_projection(lens, fmt):
    _rotating(lens, fmt, 12, 2, 512)


# 64 x 128 tiles, one slice; then slices on every tile (64 x 64, 64 x 128, 128 x 128, 256 x 128, 256 x 192), which do not divide the k-tiles but for the last
@pytest.mark.parametrize("fmt", [1, 2, 3])
@pytest.mark.parametrize("lens,Hq,Hkv,k_total", [((600, 41), 8, 2, 768), ((40, 25), 8, 2, 1792), ((33, 32), 16, 4, 2816), ((1, 65), 16, 4, 3328),
                                                 ((513, 128), 16, 4, 2816), ((256, 513), 16, 4, 4096)])
def test_rotating_projection_of_every_tile(lens, Hq, Hkv, k_total, fmt):
    _rotating(lens, fmt, Hq, Hkv, k_total // (2 if fmt == 2 else 1))


def _rotating(lens, fmt, Hq, Hkv, d):
    """The QKV projection with the rotation in its epilogue against the fp64 product and rotation."""
    print(f"feed rope {lens} fmt={fmt} heads={Hq}+{Hkv} d={d}", flush=True)
    T = sum(lens)
    heads = Hq + 2 * Hkv
    wl = W.tiny_workload("feed", 3, dtype="bf16", n_layers=1, d_model=d, n_q_heads=Hq, n_kv_heads=Hkv, head_dim=128, d_ffn=256,
                         vocab=512, block_size=16, prefix_lens=(5, 1000, 77)[:len(lens)], suffix_lens=lens)
    ctx, base = _ctx("bf16", d_model=d, n_q_heads=Hq, n_kv_heads=Hkv)
    b = W.make_batch(wl, DEV)
    bs, keep = cb.make_batch(b.suffix_ids, b.cu_suffix, b.prefix_lens, b.h_cu_suffix, b.h_prefix_lens)
    A, a64, Wt = _operands(T, heads * 128, d, fmt)
    order = torch.as_tensor(np.arange(heads * 128).reshape(heads, 4, 32)[:, [0, 2, 1, 3]].reshape(-1), device=DEV)
    out = [torch.zeros((T + 1, h, 128), dtype=torch.bfloat16, device=DEV) for h in (Hq, Hkv, Hkv)]
    ws = torch.empty(cb.confspec_workspace_bytes(ctx, T, wl.B, 0), dtype=torch.uint8, device=DEV)
    cb.confspec_op_qkv_rope(ctx, bs, 2048, A, fmt, Wt[order].contiguous(), *out, ws)
    torch.cuda.synchronize()
    a = (a64 @ f64(Wt).T).reshape(T, heads, 128)
    pos = np.concatenate([L + np.arange(S) for L, S in zip(wl.prefix_lens, wl.suffix_lens)])
    refs = (O.rope(a[:, :Hq], pos, base["rope_theta"]), O.rope(a[:, Hq:Hq + Hkv], pos, base["rope_theta"]), a[:, Hq + Hkv:])
    for got, ref in zip(out, refs):      # one rounding to 8 mantissa bits and the fp32 sum
        assert np.all(np.abs(f64(got[:T]) - ref) <= 2.0 ** -8 * np.abs(ref) + 2e-5 * np.abs(ref).max())
        assert torch.all(got[T] == 0)
    cb.confspec_destroy(ctx)


@pytest.mark.parametrize("d,F", [(2048, 6144), (2176, 6144), (4224, 4096), (6144, 16384)])
def test_reduction_with_norm_at_its_edges(d, F):
    """The kernel that adds k slices to the residual and normalises the row: 512 threads a row up to 2048 columns, 1024 above, 256 behind
    768 rows, 6144 columns the widest.  Passes of one-token traces, so that every row has a logit, against the same with no product
    split, where a kernel of its own normalises."""
    ver = None
    for rows in (100, 768, 769):
        print(f"reduction with norm d={d} F={F} rows={rows}", flush=True)
        wl = W.tiny_workload("norm", 17, dtype="bf16", n_layers=2, d_model=d, n_q_heads=8, n_kv_heads=2, head_dim=128, d_ffn=F, vocab=512, block_size=16,
                             prefix_lens=(0,) * rows, suffix_lens=(1,) * rows)
        ver = ver or Verifier(wl.model, W.make_weights(wl.model, wl.seed, DEV))
        batch = W.make_batch(wl, DEV)
        kv = W.make_seeded_kv(wl, batch, DEV)
        logits = []
        for split in (0, 1):
            cb.confspec_tune(ver.ctx, "gemm_splitk", split)
            logits.append(f64(ver.verify(kv, batch, [3, 7], [0.9])[0]))
        cb.confspec_tune(ver.ctx, "gemm_splitk", 0)
        # the two differ by the order of fp32 sums, and by the 16-bit roundings of the operands that it tips: the bound for a pass of bf16
        # operands; four columns left out of a row would move its logits by 0.04 rms
        assert np.abs(logits[0] - logits[1]).max() <= 2e-2, rows
    ver.close()
