"""The 128-wide engine of the linear backward against the oracle where it can go wrong: contractions of one to a few stages of 32 with
and without a partial last one (fewer than the ring of four is deep, exactly as many, more), ragged tiles, one split (dW and db written
by the units themselves) and several, gathered and compact rows, dX tiles of 64 and 128 rows; db alone in the same bits; several layers
in one launch."""
import re

import numpy as np
import pytest
import torch

import oracle
import paper_2210_00129_amd as sbp
import synth_inputs as si
from gpu_util import TOL_BF16_TIGHT, TOL_F32, bits, check_linear, f64, launches, nerr

pytestmark = pytest.mark.gpu
COMPACT = sbp.FLAG_DY_COMPACT | sbp.FLAG_DX_COMPACT


def _case(M, K, Cin, Cout, seed):
    idx = np.sort(np.random.default_rng(seed).choice(M, size=K, replace=False)).astype(np.int32)
    X, W, dY = si.linear_case(M, Cin, Cout, seed, "bf16")
    return X, W, dY, idx


@pytest.mark.parametrize("rows", [64, 128])
@pytest.mark.parametrize("K", [1, 31, 32, 33, 64, 97, 128, 129, 161, 2047, 2049, 4097])
def test_kept_rows_around_stages_and_splits(K, rows):
    # the dW contraction: 1 to 5 stages, the longest single split (2048 rows) and one more, two full ones and one more
    X, W, dY, idx = _case(max(2 * K, 40), K, 136, 72, K)
    with sbp.options(tile="128x128x4x64", dxrows=rows):
        check_linear(X, W, dY, idx, "bf16", flags=COMPACT if K % 2 else 0)


@pytest.mark.parametrize("rows", [64, 128])
@pytest.mark.parametrize("Cout", [8, 24, 32, 40, 64, 96, 104, 128, 136, 160, 168, 264])
def test_output_channels_around_stages(Cout, rows):
    # the dX contraction: a partial stage alone, 1 to 9 stages, partial last ones of 8, 16 and 24 channels
    X, W, dY, idx = _case(300, 131, 120, Cout, Cout)
    with sbp.options(tile="128x128x4x64", dxrows=rows):
        check_linear(X, W, dY, idx, "bf16")
        check_linear(X, W, dY, idx, "bf16", flags=sbp.FLAG_DY_COMPACT)


@pytest.mark.parametrize("K,Cin,Cout", [(40, 136, 264), (700, 264, 136), (3000, 64, 520)])
def test_db_has_the_same_bits_whichever_outputs_are_wanted(K, Cin, Cout):
    X, W, dY, idx = _case(2 * K, K, Cin, Cout, 7)
    idxd = torch.from_numpy(idx).cuda()
    Xk = sbp.forward_cache(X.cuda(), idxd)
    with sbp.options(tile="128x128x4x64"):
        full = sbp.backward_linear(dY.cuda(), idxd, Xk, W.cuda())
        alone = sbp.backward_linear(dY.cuda(), idxd, Xk, W.cuda(), want=("db",))
        with_dX = sbp.backward_linear(dY.cuda(), idxd, Xk, W.cuda(), want=("db", "dX"))
        dW0 = torch.full((Cout, Cin), 2.0, device="cuda")
        db0 = torch.full((Cout,), -1.0, device="cuda")
        acc = sbp.backward_linear(dY.cuda(), idxd, Xk, W.cuda(), flags=sbp.FLAG_ACCUMULATE_DW, dW=dW0, db=db0)
    assert np.array_equal(bits(alone[1]), bits(full[1])) and np.array_equal(bits(with_dX[1]), bits(full[1]))
    assert np.array_equal(bits(with_dX[2]), bits(full[2]))
    # accumulation adds the same sums to the old values
    assert np.array_equal(bits(acc[0]), bits(full[0] + 2.0)) and np.array_equal(bits(acc[1]), bits(full[1] - 1.0))


@pytest.mark.parametrize("K", [1, 2, 15, 16, 17, 255, 256, 257, 271, 512, 2047, 2048, 2049, 4500])
@pytest.mark.parametrize("Cout,flags", [(8, 0), (72, sbp.FLAG_DY_COMPACT), (136, 0)])
def test_db_alone_around_steps_and_batches(K, Cout, flags):
    # the column-sum blocks load 16 steps of 16 rows at a time: part of a step, one short of a batch, a whole one, one more row
    X, W, dY, idx = _case(2 * K, K, 40, Cout, K)
    idxd = torch.from_numpy(idx).cuda()
    d = dY.cuda()[idxd.long()].contiguous() if flags else dY.cuda()
    args = (d, idxd, sbp.forward_cache(X.cuda(), idxd), W.cuda())
    with sbp.options(tile="128x128x4x64"):
        full = sbp.backward_linear(*args, M=2 * K, flags=flags)
        for want in (("db",), ("db", "dX")):
            assert np.array_equal(bits(sbp.backward_linear(*args, M=2 * K, flags=flags, want=want)[1]), bits(full[1]))
    assert nerr(f64(full[1]), si.to_f64(dY)[idx].sum(0)) <= TOL_F32


def test_db_alone_of_a_gradient_beyond_4_GB():
    # row offsets that need more than 32 bits
    M, Cout, K = 2_200_000, 1000, 300
    dY = torch.empty((M, Cout), dtype=torch.bfloat16, device="cuda")
    idx = np.sort(np.random.default_rng(5).choice(M - 1, size=K - 1, replace=False)).astype(np.int32)
    idxd = torch.from_numpy(np.append(idx, M - 1).astype(np.int32)).cuda()
    rows = torch.randn((K, Cout)).to(torch.bfloat16)
    dY[idxd.long()] = rows.cuda()
    db = sbp.backward_linear(dY, idxd, None, torch.empty((Cout, 8), dtype=torch.bfloat16, device="cuda"), want=("db",))[1]
    assert nerr(f64(db), si.to_f64(rows).sum(0)) <= TOL_F32


def test_layers_of_one_launch_longest_workgroups_first():
    # four layers whose kinds of workgroups differ in length by an order of magnitude, one of them without dX, one compact, one
    # accumulating: the launch orders their segments by length, whatever the layer
    shapes = [(900, 136, 1048, 0, True), (64, 72, 40, COMPACT, True), (1800, 264, 136, sbp.FLAG_ACCUMULATE_DW, True), (130, 520, 8, 0, False)]
    layers, refs = [], []
    for i, (K, Cin, Cout, flags, want_dx) in enumerate(shapes):
        M = 2 * K
        X, W, dY, idx = _case(M, K, Cin, Cout, 40 + i)
        idxd = torch.from_numpy(idx).cuda()
        refs.append(oracle.backward_linear(si.to_f64(dY), idx, si.to_f64(X)[idx], si.to_f64(W), M) + (idx,))
        d = dY.cuda()[idxd.long()].contiguous() if flags & sbp.FLAG_DY_COMPACT else dY.cuda()
        l = dict(dY=d, idx=idxd, X_k=sbp.forward_cache(X.cuda(), idxd), W=W.cuda(), M=M, flags=flags,
                 dW=torch.full((Cout, Cin), 1.0, device="cuda"), db=torch.full((Cout,), 1.0, device="cuda"))
        if want_dx:
            l["dX"] = torch.full((K if flags & sbp.FLAG_DX_COMPACT else M, Cin), 9.0, dtype=torch.bfloat16, device="cuda")
        layers.append(l)
    out = sbp.backward_linear_batch(layers, want=())
    torch.cuda.synchronize()
    for (K, Cin, Cout, flags, want_dx), l, (rW, rb, rX, idx) in zip(shapes, layers, refs):
        one = 1.0 if flags & sbp.FLAG_ACCUMULATE_DW else 0.0
        assert nerr(f64(l["dW"]), rW + one) <= TOL_F32 and nerr(f64(l["db"]), rb + one) <= TOL_F32
        if want_dx:
            assert nerr(f64(l["dX"]), rX[idx] if flags & sbp.FLAG_DX_COMPACT else rX) <= TOL_BF16_TIGHT


@pytest.mark.parametrize("dxrows", [None, 64, 128])
@pytest.mark.parametrize("order", [None, "0,1,2", "2,0,1", "1,2,0"])
def test_batch_in_one_launch_follows_the_overrides(dxrows, order, capfd):
    # three layers, one split and several, one of them without dX: one launch, its segments by length or by the kinds' order given by
    # hand, dX tiles as given by hand; every choice with the bits of dX and dW that the oracle bounds
    shapes = [(500, 136, 264, True), (1800, 264, 136, True), (700, 72, 520, False)]
    layers, refs = [], []
    for i, (K, Cin, Cout, want_dx) in enumerate(shapes):
        X, W, dY, idx = _case(2 * K, K, Cin, Cout, 60 + i)
        idxd = torch.from_numpy(idx).cuda()
        refs.append(oracle.backward_linear(si.to_f64(dY), idx, si.to_f64(X)[idx], si.to_f64(W), 2 * K))
        layers.append(dict(dY=dY.cuda(), idx=idxd, X_k=sbp.forward_cache(X.cuda(), idxd), W=W.cuda(), M=2 * K,
                           inv=torch.from_numpy(oracle.inverse_map(idx, 2 * K)).cuda(), dW=torch.empty((Cout, Cin), device="cuda"),
                           db=torch.empty((Cout,), device="cuda")))
        if want_dx:
            layers[-1]["dX"] = torch.empty((2 * K, Cin), dtype=torch.bfloat16, device="cuda")
    opts = {k: v for k, v in dict(dxrows=dxrows, order=order).items() if v}
    with sbp.options(debug_plan=1, **opts):
        n = launches(lambda: sbp.backward_linear_batch(layers, want=()))
    assert n["dw_gemm"] == 1 and n["reduce"] == 1
    text = [line for line in capfd.readouterr().err.splitlines() if line.startswith("sbp batch of 128-wide tiles:")][-1]
    segments = [(int(l), int(k), float(us)) for l, k, us in re.findall(r"L(\d)\.k(\d) \d+ x ([\d.]+)us", text)]
    assert sorted((l, k) for l, k, _ in segments) == [(0, 0), (0, 1), (0, 2), (1, 0), (1, 1), (1, 2), (2, 1)]
    kinds = [k for _, k, _ in segments]
    if order:
        assert kinds == sorted(kinds, key=[int(k) for k in order.split(",")].index)
    for (_, k0, a), (_, k1, b) in zip(segments, segments[1:]):
        assert a >= b or (order and k0 != k1)
    rows = [int(r) for r in re.findall(r"dx rows (\d+)", text)]
    assert len(rows) == 3 and (not dxrows or set(rows) == {dxrows})
    for l, k, us in segments:                          # the lengths are the planner's: 4 us + 0.3 us per stage of 32 (64 rows: 0.21)
        if k == 0:
            assert abs(us - (4 + (0.21 if rows[l] == 64 else 0.3) * -(-shapes[l][2] // 32))) <= 0.06
    for l, (rW, rb, rX), (_, _, _, want_dx) in zip(layers, refs, shapes):
        assert nerr(f64(l["dW"]), rW) <= TOL_F32 and nerr(f64(l["db"]), rb) <= TOL_F32
        if want_dx:
            assert nerr(f64(l["dX"]), rX) <= TOL_BF16_TIGHT


@pytest.mark.parametrize("opts", [dict(dxrows=64, tile="128x128x4x64"), dict(dxrows=128, tile="128x128x4x64"), dict(tile="256x256x8x64"),
                                  dict(tile="256x256x4x32")])
@pytest.mark.parametrize("Cout", [8, 40, 72, 120, 200])
def test_infinite_gradients_in_the_last_partial_stage(Cout, opts):
    # dX of a row with an infinite gradient is infinite where its weight is not zero, never NaN: the last, partial stage of the
    # contraction over Cout holds copies of the row's last 8 channels, which must count for nothing
    X, W, dY, idx = _case(300, 131, 120, Cout, Cout + 1)
    rows = torch.from_numpy(idx[::7]).long()
    dY[rows, Cout - 1 - (rows % 8)] = float("inf")
    W[W == 0] = 0.01
    idxd = torch.from_numpy(idx).cuda()
    with sbp.options(**opts):
        dX = sbp.backward_linear(dY.cuda(), idxd, None, W.cuda(), want=("dX",))[2]
    got = dX.cpu().double()[torch.from_numpy(idx).long()]
    ref = dY.double()[torch.from_numpy(idx).long()] @ W.double()
    assert torch.isinf(ref).any() and not torch.isnan(ref).any()
    fin = torch.isfinite(ref)
    assert torch.equal(got[~fin], ref[~fin])
    assert nerr(got[fin].numpy(), ref[fin].numpy()) <= TOL_BF16_TIGHT


@pytest.mark.parametrize("K", [33, 40, 41, 57, 1001])
@pytest.mark.parametrize("tile", ["128x128x4x64", "big"])
def test_infinite_cached_values_in_the_last_row_group(K, tile):
    # the same for dW with X_k in row groups: whole groups past the last row hold copies of the last group
    X, W, dY, idx = _case(2 * K, K, 136, 96, K)
    last = int(idx[-1])
    X[last, 5] = float("inf")
    dY[last][dY[last] == 0] = 0.5
    idxd = torch.from_numpy(idx).cuda()
    (Xt,) = sbp.forward_cache_batch([X.cuda()], [idxd], layout=sbp.LAYOUT_KMAJOR)
    with sbp.options(tile=tile):
        dW = sbp.backward_linear(dY.cuda(), idxd, Xt, W.cuda(), flags=sbp.FLAG_XK_KMAJOR, want=("dW",))[0].cpu().double()
    rows = torch.from_numpy(idx).long()
    ref = dY.double()[rows].T @ X.double()[rows]
    fin = torch.isfinite(ref)
    assert torch.equal(dW[~fin], ref[~fin]) and not fin[:, 5].any() and fin[:, 6:].all()
    assert nerr(dW[fin].numpy(), ref[fin].numpy()) <= TOL_F32


@pytest.mark.parametrize("K,Cin,Cout", [(1500, 2048, 1536), (3000, 256, 3072), (1584, 768, 2304), (2100, 1024, 3072)])
@pytest.mark.parametrize("want", [("dW",), ("dW", "db"), ("db",)])
def test_calls_without_dX_take_the_128_wide_tiles(K, Cin, Cout, want):
    # layers whose full call takes (or took) the large tiles: the engines sum in different orders, so the bits tell which one ran; the
    # workspace is the one that is asked for without knowing the wanted outputs
    X, W, dY, idx = _case(K + 64, K, Cin, Cout, K)
    idxd = torch.from_numpy(idx).cuda()
    args = (dY.cuda(), idxd, sbp.forward_cache(X.cuda(), idxd), W.cuda())
    ws = torch.empty(max(256, sbp.backward_linear_workspace(K + 64, K, Cin, Cout, sbp.BF16)), dtype=torch.uint8, device="cuda")
    out = sbp.backward_linear(*args, want=want, workspace=ws)
    forced = {}
    for tile in ("128x128x4x64", "big"):
        with sbp.options(tile=tile):
            forced[tile] = sbp.backward_linear(*args, want=want)
    for a, b, c in zip(out[:2], forced["128x128x4x64"], forced["big"]):
        if a is not None:
            assert np.array_equal(bits(a), bits(b)) and not np.array_equal(bits(a), bits(c))
            assert nerr(f64(a), f64(c)) <= 2 * TOL_F32
