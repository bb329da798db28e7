"""The fp32 matrix-core kernel of the linear backward (fp32 tensors, odd channel counts, unaligned tensors) at the edges of
its tiles, stages (64 each) and splits, against the oracle.  Bounds: fp32 sums of exact or singly rounded products, in chains
of at most 256 rows, stay below 1e-5 of max |result|; dX of bf16 tensors is rounded once (gpu_util)."""
import numpy as np
import pytest
import torch

import oracle
import paper_2210_00129_amd as sbp
import synth_inputs as si
from gpu_util import TOL_BF16_TIGHT, TOL_F32, bits, check_linear, f64, launches, nerr

pytestmark = pytest.mark.gpu


def _rows(M, K, seed=3):
    return np.random.default_rng(seed).permutation(M)[:K].astype(np.int32)


# (K, Cin, Cout): one row; one short of, at and one past a stage and a tile; several splits; pieces of 4 and single elements
SIZES = [(1, 4, 4), (1, 1, 1), (31, 64, 32), (32, 60, 64), (33, 68, 96), (64, 128, 65), (65, 63, 128), (257, 7, 130),
         (700, 64, 260), (1500, 132, 36), (3000, 66, 190)]


@pytest.mark.parametrize("K,Cin,Cout", SIZES)
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_tile_stage_and_split_edges(K, Cin, Cout, dtype):
    if dtype == "bf16" and Cin % 8 == 0 and Cout % 8 == 0:
        Cin += 3                                             # (multiples of 8 go to the bf16 engines)
    M = K + K // 2 + 5
    X, W, dY = si.linear_case(M, Cin, Cout, 11, dtype)
    idx = _rows(M, K)
    check_linear(X, W, dY, idx, dtype)
    check_linear(X, W, dY, idx, dtype, flags=sbp.FLAG_DY_COMPACT | sbp.FLAG_DX_COMPACT, check_cache=False)


@pytest.mark.parametrize("K,Cin,Cout", [(21900, 260, 132), (21801, 259, 130)])
def test_more_units_than_fit_at_once(K, Cin, Cout):
    # several rounds of workgroups, in pieces of 4 and in single elements
    M = K + 777
    X, W, dY = si.linear_case(M, Cin, Cout, 12, "f32")
    check_linear(X, W, dY, _rows(M, K), "f32", inv_mode="sampler")


@pytest.mark.parametrize("want", [("db",), ("dX",), ("dW",), ("dW", "db"), ("db", "dX")])
@pytest.mark.parametrize("K", [100, 2000, 20000])            # one split (dW and db written directly) and several; 64 slices of db alone
def test_single_outputs_and_accumulation(want, K):
    M, Cin, Cout = K + 50, 72, 200
    X, W, dY = si.linear_case(M, Cin, Cout, 13, "f32")
    idx_np = _rows(M, K)
    idx = torch.from_numpy(idx_np).cuda()
    Xk = X[idx.cpu().long()].cuda()
    ref = dict(zip(("dW", "db", "dX"), oracle.backward_linear(si.to_f64(dY), idx_np, si.to_f64(X)[idx_np], si.to_f64(W), M)))
    for flags in (0, sbp.FLAG_ACCUMULATE_DW):
        out = {}
        if flags:
            out = {n: torch.ones(s, device="cuda") for n, s in (("dW", (Cout, Cin)), ("db", (Cout,))) if n in want}
        got = dict(zip(("dW", "db", "dX"), sbp.backward_linear(dY.cuda(), idx, Xk, W.cuda(), want=want, flags=flags, **out)))
        torch.cuda.synchronize()
        for n in ("dW", "db", "dX"):
            assert (got[n] is not None) == (n in want)
            if n in want:
                assert nerr(f64(got[n]), ref[n] + (1 if flags and n != "dX" else 0)) <= TOL_F32, (n, flags)


def test_unaligned_bf16_tensors_of_a_large_layer():
    # sizes that plan the 256-wide bf16 engine, addresses that rule it out
    M, K, Cin, Cout = 3000, 2100, 256, 512
    X, W, dY = si.linear_case(M, Cin, Cout, 14, "bf16")
    idx_np = _rows(M, K)
    shift = lambda t: torch.empty(t.numel() + 1, dtype=t.dtype, device="cuda")[1:].view(t.shape).copy_(t)
    idx = torch.from_numpy(idx_np).cuda()
    dW, db, dX = sbp.backward_linear(shift(dY), idx, shift(X[torch.from_numpy(idx_np).long()]), shift(W))
    torch.cuda.synchronize()
    rW, rb, rX = oracle.backward_linear(si.to_f64(dY), idx_np, si.to_f64(X)[idx_np], si.to_f64(W), M)
    assert nerr(f64(dW), rW) <= TOL_F32 and nerr(f64(db), rb) <= TOL_F32 and nerr(f64(dX), rX) <= TOL_BF16_TIGHT
    assert np.all(bits(dX)[np.setdiff1d(np.arange(M), idx_np)] == 0)


@pytest.mark.parametrize("K,Cin,Cout,dtype", [(9000, 2048, 2048, "f32"), (16384, 768, 772, "f32"), (12000, 1023, 2049, "f32"),
                                              (30000, 1021, 1031, "bf16"), (12000, 1028, 2052, "bf16"),
                                              (20000, 2048, 2052, "f32"), (20000, 2049, 2051, "f32"), (20000, 2052, 2052, "bf16"),
                                              (20000, 2049, 2049, "bf16")])
def test_long_splits_are_summed_in_short_chains(K, Cin, Cout, dtype):
    # splits of 2000 to 20000 rows, single ones written directly.  A running sum of n zero-mean products ends up off by
    # u sqrt(n / 6) of its size (u = 2^-24: n additions, each off by up to half a unit of the last place of a partial sum that
    # grows as sqrt(i)); chains of at most 256 rows, at most 128 of them or in a compensated sum, then
    # up to 64 splits: n = 256 + 64
    g = torch.Generator(device="cuda").manual_seed(7)
    X, dY = (torch.randn(K, c, generator=g, device="cuda").to(si.torch_dtype(dtype)) for c in (Cin, Cout))
    W = torch.randn(Cout, Cin, generator=g, device="cuda").to(si.torch_dtype(dtype))
    idx = torch.randperm(K, generator=g, device="cuda").int()
    engine, splits = sbp.backward_linear_engine(K, K, Cin, Cout, sbp.F32 if dtype == "f32" else sbp.BF16)
    assert engine == "plain" and K // splits > 2000
    dW, db, _ = sbp.backward_linear(dY, idx, X, W, want=("dW", "db"))
    alone = sbp.backward_linear(dY, idx, X, W, want=("db",))[1]
    G = dY.double()[idx.long()]
    rW, rb = torch.matmul(G.t().contiguous(), X.double()), G.sum(0)
    bound = 2.0 ** -24 * (320 / 6) ** 0.5
    for got, want in ((dW, rW), (db, rb), (alone, rb)):
        assert ((got.double() - want).norm() / want.norm()).item() <= bound


@pytest.mark.parametrize("K,Cin,Cout", [(900, 200, 1000), (2100, 640, 264), (16800, 136, 256), (130, 72, 40)])
@pytest.mark.parametrize("off", ["dY", "X_k", "W"])
def test_unaligned_bf16_tensors_have_splits_of_their_own(K, Cin, Cout, off):
    # a tensor one element off 16 bytes sends a bf16 layer to the fp32 engine, whose units are smaller than those of the bf16 ones: it
    # cuts dW by a rule of its own (several splits from 512 rows on where the layer is small), in the workspace of the bf16 plan
    M = K + 40
    X, W, dY = si.linear_case(M, Cin, Cout, 17, "bf16")
    idx_np = _rows(M, K)

    def put(t, name):
        flat = torch.empty(t.numel() + 1, dtype=t.dtype, device="cuda")
        view = flat[1:] if name == off else flat[:-1]
        return view.view(t.shape).copy_(t)
    idx = torch.from_numpy(idx_np).cuda()
    dYd, Xk, Wd = put(dY, "dY"), put(X[torch.from_numpy(idx_np).long()], "X_k"), put(W, "W")
    ref = oracle.backward_linear(si.to_f64(dY), idx_np, si.to_f64(X)[idx_np], si.to_f64(W), M)
    for flags in (0, sbp.FLAG_DW_OUT_BF16):
        dW, db, dX = sbp.backward_linear(dYd, idx, Xk, Wd, flags=flags)
        assert nerr(f64(dW), ref[0]) <= (TOL_BF16_TIGHT if flags else TOL_F32) and nerr(f64(db), ref[1]) <= TOL_F32
        assert nerr(f64(dX), ref[2]) <= TOL_BF16_TIGHT
    n = launches(lambda: sbp.backward_linear(dYd, idx, Xk, Wd, want=("dW",)))
    assert n["dw_gemm"] == 1 and n["reduce"] == (1 if K > 256 else 0)
