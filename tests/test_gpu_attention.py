"""GPU parity of the attention backward on the kept tokens ("Drop QKV") against the fp64 oracle, through
the C ABI.  The forward (attention output and the row log-sum-exp over all keys) is the model's, computed
by the library routines of the input module; the oracle gets the full q, k, v and the keep sets, the HIP
path only the kept rows."""
import math
import os

import numpy as np
import pytest
import torch

import oracle
import paper_2210_00129_amd as sbp
import synth_inputs as si
from gpu_util import TOL_BF16, TOL_F32, f64, nerr

pytestmark = pytest.mark.gpu


def _keep_sets(B, n, n_k, seed):
    g = np.random.default_rng(seed)
    return np.stack([np.sort(g.choice(n, size=n_k, replace=False)) for _ in range(B)])


def _run(B, n, h, d, keep, dtype, seed, scale=None):
    scale = 1.0 / math.sqrt(d) if scale is None else scale
    n_k = keep.shape[1]
    qkv, dA = si.attention_case(B, n, h, d, seed, dtype)
    A64, lse64 = si.attention_forward(qkv, B, n, h, d, scale)
    tdt = si.torch_dtype(dtype)
    A = A64.to(tdt)                                   # a forward stores its output in the model's type
    lse = lse64.to(torch.float32)
    rows = torch.from_numpy((np.arange(B)[:, None] * n + keep).reshape(-1)).long()
    dA_k = dA[rows].contiguous()
    out = sbp.backward_attention(qkv[rows].contiguous().cuda(), A[rows].contiguous().cuda(), dA_k.cuda(),
                                 lse[rows].contiguous().cuda(), B, h, d, scale)
    torch.cuda.synchronize()
    x = si.to_f64(qkv).reshape(B, n, 3, h, d)
    ref = oracle.backward_attention(si.to_f64(dA_k).reshape(B, n_k, h, d), x[:, :, 0], x[:, :, 1], x[:, :, 2], keep, scale)
    got = f64(out).reshape(B, n_k, 3, h, d)
    return [nerr(got[:, :, i], ref[i]) for i in range(3)]


CASES = [  # B, n, h, d, n_k
    (2, 197, 3, 64, 99),      # ViT at r = 0.5: 4 blocks of 32 with a ragged tail
    (1, 197, 2, 64, 197),     # everything kept: 7 blocks
    (2, 50, 2, 64, 1),        # a single kept token
    (2, 70, 2, 64, 32),       # exactly one block
    (1, 70, 1, 64, 33),
    (1, 300, 1, 64, 256),     # two full chunks (the most that one workgroup per head could hold at d = 64)
    (1, 300, 1, 64, 257),     # one more: three chunks, the last with one token
    (1, 600, 2, 64, 512),     # four full chunks
    (1, 1100, 1, 64, 1024),
    (1, 400, 1, 32, 390),
    (1, 300, 1, 128, 161),
    (2, 120, 3, 32, 100),
    (1, 140, 2, 128, 100),
    (2, 40, 2, 16, 21),       # d = 16: plain kernel
]


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("B,n,h,d,n_k", CASES)
def test_attention_backward_matches_oracle(B, n, h, d, n_k, dtype):
    errs = _run(B, n, h, d, _keep_sets(B, n, n_k, 5), dtype, 3)
    tol = TOL_F32 if dtype == "f32" else TOL_BF16
    assert max(errs) <= tol, errs


def test_engine_choice():
    assert sbp.backward_attention_engine(64, 64, sbp.BF16) == "mfma"
    assert sbp.backward_attention_engine(99, 64, sbp.BF16) == "mfma_tiled"
    assert sbp.backward_attention_engine(257, 64, sbp.BF16) == "mfma_tiled"
    assert sbp.backward_attention_engine(4096, 128, sbp.BF16) == "mfma_tiled"
    assert sbp.backward_attention_engine(99, 64, sbp.F32) == "mfma_f32"
    assert sbp.backward_attention_engine(99, 16, sbp.BF16) == "plain"


def test_plain_kernel_on_bf16_matches_oracle():
    with sbp.options(attn="plain"):
        assert sbp.backward_attention_engine(99, 64, sbp.BF16) == "plain"
        errs = _run(2, 197, 3, 64, _keep_sets(2, 197, 99, 7), "bf16", 9)
    assert sbp.backward_attention_engine(99, 64, sbp.BF16) == "mfma_tiled"
    assert max(errs) <= TOL_BF16, errs


def test_grid_sampler_keep_sets_and_other_scale():
    # keep sets as the library's sampler draws them (class token + 2x2 grid cells), a non-default scale
    B, P, H, W, h, d = 3, 1, 14, 14, 2, 64
    n = P + H * W
    idx = sbp.sample_indices(B, P, H, W, 2, 17, 4)[0].cpu().numpy().astype(np.int64)
    n_k = idx.size // B
    keep = (idx.reshape(B, n_k) - np.arange(B)[:, None] * n)
    assert keep.min() >= 0 and keep.max() < n
    errs = _run(B, n, h, d, keep, "bf16", 21, scale=0.09)
    assert max(errs) <= TOL_BF16, errs


def test_bench_size_vit_base():
    # the size bench.py times: B = 64, 12 heads of 64, 99 of 197 tokens kept
    B, n, h, d, n_k = 64, 197, 12, 64, 99
    errs = _run(B, n, h, d, _keep_sets(B, n, n_k, 1), "bf16", 2)
    assert max(errs) <= TOL_BF16, errs


def test_feeds_the_qkv_linear_backward():
    # dqkv_k is the compact dY of the qkv projection: its backward from these rows equals the oracle's
    B, n, h, d, n_k, C = 2, 50, 2, 64, 25, 64
    keep = _keep_sets(B, n, n_k, 3)
    scale = 1.0 / math.sqrt(d)
    qkv, dA = si.attention_case(B, n, h, d, 4, "bf16")
    A64, lse64 = si.attention_forward(qkv, B, n, h, d, scale)
    rows_np = (np.arange(B)[:, None] * n + keep).reshape(-1)
    rows = torch.from_numpy(rows_np).long()
    X, Wt, _ = si.linear_case(B * n, C, 3 * h * d, 6, "bf16")
    dqkv = sbp.backward_attention(qkv[rows].contiguous().cuda(), A64.to(torch.bfloat16)[rows].contiguous().cuda(),
                                  dA[rows].contiguous().cuda(), lse64.float()[rows].contiguous().cuda(), B, h, d, scale)
    idx = torch.from_numpy(rows_np.astype(np.int32)).cuda()
    Xk = sbp.forward_cache(X.cuda(), idx)
    dW, db, dX = sbp.backward_linear(dqkv, idx, Xk, Wt.cuda(), M=B * n, flags=sbp.FLAG_DY_COMPACT)
    torch.cuda.synchronize()
    dY_full = np.zeros((B * n, 3 * h * d))
    dY_full[rows_np] = f64(dqkv)                      # the same rounded rows the kernel consumed
    rW, rb, rX = oracle.backward_linear(dY_full, rows_np, si.to_f64(X)[rows_np], si.to_f64(Wt), B * n)
    assert nerr(f64(dW), rW) <= TOL_F32 and nerr(f64(db), rb) <= TOL_F32 and nerr(f64(dX), rX) <= TOL_BF16


def test_empty_and_errors():
    e = torch.empty((0, 3 * 2 * 64), dtype=torch.bfloat16, device="cuda")
    a = torch.empty((0, 2 * 64), dtype=torch.bfloat16, device="cuda")
    l = torch.empty((0, 2), dtype=torch.float32, device="cuda")
    assert sbp.backward_attention(e, a, a, l, 1, 2, 64, 0.125).shape == (0, 384)
    q = torch.zeros((4, 3 * 2 * 24), dtype=torch.bfloat16, device="cuda")
    with pytest.raises(Exception):
        sbp.backward_attention(q, q[:, :48], q[:, :48], torch.zeros((4, 2), device="cuda"), 1, 2, 24, 0.2)   # d = 24


@pytest.mark.parametrize("B,n,h,d,n_k", [(2, 197, 3, 64, 99), (1, 197, 2, 64, 197), (2, 50, 2, 64, 1), (1, 70, 1, 64, 33),
                                         (1, 300, 1, 64, 256), (2, 120, 3, 32, 100), (1, 140, 2, 128, 100)])
def test_tiled_kernel_at_sizes_the_single_workgroup_kernel_also_serves(B, n, h, d, n_k):
    # the two matrix-core kernels do the same products on the same rounded probabilities: both within the bar, and
    # close to each other
    keep = _keep_sets(B, n, n_k, 11)
    with sbp.options(attn="tiled"):
        assert sbp.backward_attention_engine(n_k, d, sbp.BF16) == "mfma_tiled"
        errs = _run(B, n, h, d, keep, "bf16", 13)
    assert max(errs) <= TOL_BF16, errs
    with sbp.options(attn="whole"):
        assert sbp.backward_attention_engine(n_k, d, sbp.BF16) == "mfma"
        errs_w = _run(B, n, h, d, keep, "bf16", 13)
    assert max(errs_w) <= TOL_BF16, errs_w


@pytest.mark.parametrize("d", [32, 64, 128])
@pytest.mark.parametrize("n_k", [31, 64, 65, 128, 129])
def test_f32_matrix_core_kernel_at_tile_and_chunk_edges(d, n_k):
    # streamed tiles of 32 tokens, chunks of 128 owned per workgroup; the plain kernel stays behind the option
    keep = _keep_sets(2, 160, n_k, 23)
    assert max(_run(2, 160, 2, d, keep, "f32", 25)) <= TOL_F32
    with sbp.options(attn="plain"):
        assert max(_run(2, 160, 2, d, keep, "f32", 25)) <= TOL_F32


@pytest.mark.parametrize("d", [32, 64, 128])
@pytest.mark.parametrize("n_k", [64, 65, 129, 577])
def test_bf16_dispatch_edge_and_table_refill(d, n_k):
    # 64 tokens: the last size of the one-workgroup kernel; 65: a tile of 64 and one row; 129: a second chunk of one token;
    # 577: the tables of queries 512 .. are made inside the loop, then one more row behind a full tile
    assert max(_run(1, 600, 2, d, _keep_sets(1, 600, n_k, 27), "bf16", 29)) <= TOL_BF16


@pytest.mark.parametrize("n_k", [896, 897, 1024, 1100])
def test_bf16_table_refills_of_short_heads(n_k):
    # d = 32, tables of 512 queries refilled inside the loop: 384 queries in the second table, one more, a full one, a third
    assert max(_run(1, 1100, 2, 32, _keep_sets(1, 1100, n_k, 31), "bf16", 33)) <= TOL_BF16


def test_f32_more_heads_than_one_grid_of_the_matrix_core_kernel_holds():
    # two workgroups of 256 threads per head: 2^23 heads would be a grid of 2^32 threads, from there on the plain kernel runs
    B, h, d, n_k = 65535, 129, 32, 3
    g = torch.Generator(device="cuda").manual_seed(3)
    qkv = torch.randn(B * n_k, 3 * h * d, generator=g, device="cuda")
    dA = torch.randn(B * n_k, h * d, generator=g, device="cuda")
    A = torch.zeros_like(dA)
    lse = torch.zeros(B * n_k, h, device="cuda")
    some = [(0, 0), (0, h - 1), (B // 2, 64), (B - 1, 0), (B - 1, h - 1)]
    want = []
    for b, head in some:
        rows, c = slice(b * n_k, (b + 1) * n_k), slice(head * d, (head + 1) * d)
        q, k, v = (qkv[rows, i * h * d + head * d:i * h * d + (head + 1) * d].double() for i in range(3))
        s = torch.matmul(q, k.t().contiguous()) * d ** -0.5
        lse[rows, head] = torch.logsumexp(s, -1).float()
        P = torch.softmax(s, -1)
        A[rows, c] = torch.matmul(P, v).float()
        G = dA[rows, c].double()
        dS = P * (torch.matmul(G, v.t().contiguous()) - (G * A[rows, c].double()).sum(-1, keepdim=True))
        want.append([torch.matmul(dS, k) * d ** -0.5, torch.matmul(dS.t().contiguous(), q) * d ** -0.5, torch.matmul(P.t().contiguous(), G)])
    out = torch.full_like(qkv, float("nan"))
    sbp.backward_attention(qkv, A, dA, lse, B, h, d, d ** -0.5, out=out)
    for (b, head), w in zip(some, want):
        for i in range(3):
            got = out[b * n_k:(b + 1) * n_k, i * h * d + head * d:i * h * d + (head + 1) * d]
            assert nerr(f64(got), f64(w[i])) <= TOL_F32
    assert not torch.isnan(out).any()


@pytest.mark.parametrize("d", [32, 64, 128])
@pytest.mark.parametrize("B,h", [(2, 2), (40, 8)])
@pytest.mark.parametrize("n_k", [1, 2, 3, 4, 5, 16, 17])
def test_f32_heads_of_a_few_tokens(B, h, d, n_k):
    # the plain kernel up to 2, 4, 16 tokens (1, 2, 4 where there are few heads), the matrix cores beyond: the same gradients
    assert max(_run(B, 20, h, d, _keep_sets(B, 20, n_k, 35), "f32", 37)) <= TOL_F32
    few = {32: 2, 64: 4, 128: 16}[d]
    assert sbp.backward_attention_engine(n_k, d, sbp.F32) == ("plain" if n_k <= few else "mfma_f32")
