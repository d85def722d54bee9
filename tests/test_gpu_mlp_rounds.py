"""The rows kernel of the sparse MLP at the edges of its launch rules: row
counts on both sides of the 2- and 4-row rounds and of the row teams that
narrow rows get, one- and two-vector slices over 1 to 16 waves in each type,
more rows per workgroup than its threads load in one pass, and a row without
a slot under an infinite x.  Records and x are dyadic (m 2^-6, |m| <= 1; x in
{-1, 0, 1}), so every sum is exact in fp32 in any order and y must equal the
oracle's value for value."""
import numpy as np
import pytest
import torch

import oracle as orc
from paper_2608_22643_amd import binding as B
from paper_2608_22643_amd import workload as W
from gpu_util import DEV, Bufs, decode_y, say, to_dev

pytestmark = pytest.mark.gpu

# (d, type, row counts, workgroups forced through NP_MLP_WG or None)
CASES = [
    (256, "f32", (3, 511, 512, 513), None),             # 1 wave, 2- and 4-row rounds
    (264, "f16", (1023, 1024, 2047, 2048, 2051), None),  # 1 wave: 1, 2 and 4 teams, ragged width
    (1000, "bf16", (511, 1023, 1024, 1500), None),       # 2 waves: 1 and 2 teams
    (2048, "f32", (512, 1030), None),                    # 8 waves of one vector
    (2568, "f32", (512, 600), None),                     # 6 waves of two vectors
    (4608, "f16", (9, 517), None),                       # 9 waves
    (8192, "bf16", (511, 1027), None),                   # 8 waves of two vectors
    (8192, "f32", (257, 515), None),                     # 16 waves of two vectors
    (16384, "bf16", (2, 513), None),                     # 16 waves of two vectors
    (512, "f16", (1100, 1600), 1),                       # a range longer than the workgroup
]


@pytest.mark.parametrize("d,dt,rows,wg", CASES, ids=[f"d{c[0]}_{c[1]}" for c in CASES])
def test_mlp_rounds_exact(d, dt, rows, wg, monkeypatch):
    if wg:
        monkeypatch.setenv("NP_MLP_WG", str(wg))
    k = max(rows)
    F, C = k + 40, k + 20
    cfg = W.Config("rounds", 1, d, F, 8, k / F, C / F, dt, dt, 1, rho_given=0.0, k_override=k,
                   c_override=C, dyadic=True, dyadic_w_range=1, dyadic_h_range=1)
    say(f"[mlp rounds] d {d} {dt} rows {rows}")
    bufs = Bufs(cfg)
    bufs.reset()
    rng = np.random.default_rng(d + k)
    store, h = W.storage(cfg), W.hidden(cfg, 1)[0]
    neuron = rng.permutation(F)[:C].astype(np.int32)
    res, x = to_dev(store[0][neuron]), to_dev(h)
    slots = rng.permutation(C)[:k].astype(np.int32)
    y = torch.zeros(d * W.ITEMSIZE[dt], dtype=torch.uint8, device=DEV)
    xv = orc.decode(dt, h)
    rec = orc.decode(dt, store[0][neuron[slots]])
    a = np.maximum(rec[:, :d] @ xv, 0) * (rec[:, d:2 * d] @ xv)
    assert np.max(np.abs(a)) < 2.0 ** 12 and np.max(np.abs(a) @ np.abs(rec[:, 2 * d:])) < 2.0 ** 6
    for n in rows:
        B.np_sparse_mlp(bufs.shape, 0, x, res, to_dev(slots), n, y, bufs.ws)
        torch.cuda.synchronize()
        ref = orc.sparse_mlp(cfg, 0, h, store, neuron[slots[:n]])
        assert np.array_equal(decode_y(orc, dt, y.cpu().numpy()), decode_y(orc, dt, ref)), n
    # the dense call: every record of one layer, in order
    B.np_dense_mlp(bufs.shape, to_dev(store[0]), x, y, bufs.ws)
    torch.cuda.synchronize()
    ref = orc.sparse_mlp(cfg, 0, h, store, np.arange(F, dtype=np.int32))
    assert np.array_equal(decode_y(orc, dt, y.cpu().numpy()), decode_y(orc, dt, ref)), "dense"
    assert B.np_device_error(bufs.ws) == 0
    # rows without a slot add nothing, also where x is infinite
    bad = np.full(k, -1, np.int32)
    bad[::2] = C + 3
    inf = torch.full((d,), float("inf"), dtype={"f32": torch.float32, "f16": torch.float16,
                                                "bf16": torch.bfloat16}[dt], device=DEV)
    B.np_sparse_mlp(bufs.shape, 0, inf, res, to_dev(bad), k, y, bufs.ws)
    torch.cuda.synchronize()
    assert np.all(decode_y(orc, dt, y.cpu().numpy()) == 0)
    assert B.np_device_error(bufs.ws) == B.NP_DEVERR_NOT_RESIDENT


# (d, type, rows, NP_MLP_R, NP_MLP_TEAMS): forced rounds and teams that the
# rule does not take by itself
KNOBS = [
    (256, "f32", 700, 2, 4), (264, "f16", 300, 4, 4), (1000, "bf16", 1030, 2, 4),
    (2048, "f16", 515, 4, 2), (4096, "f16", 1030, 2, 2), (5120, "f16", 523, 2, 2),
    (5120, "bf16", 2051, 4, 1), (8192, "bf16", 259, 4, 2),
]


@pytest.mark.parametrize("d,dt,n,R,teams", KNOBS, ids=[f"d{c[0]}_{c[1]}_R{c[3]}_T{c[4]}" for c in KNOBS])
def test_mlp_forced_rounds_and_teams_exact(d, dt, n, R, teams, monkeypatch):
    monkeypatch.setenv("NP_MLP_R", str(R))
    monkeypatch.setenv("NP_MLP_TEAMS", str(teams))
    F, C = n + 40, n + 20
    cfg = W.Config("forced", 1, d, F, 8, n / F, C / F, dt, dt, 1, rho_given=0.0, k_override=n,
                   c_override=C, dyadic=True, dyadic_w_range=1, dyadic_h_range=1)
    say(f"[mlp forced] d {d} {dt} rows {n} R {R} teams {teams}")
    bufs = Bufs(cfg)
    bufs.reset()
    rng = np.random.default_rng(d + n)
    store, h = W.storage(cfg), W.hidden(cfg, 1)[0]
    neuron = rng.permutation(F)[:C].astype(np.int32)
    slots = rng.permutation(C)[:n].astype(np.int32)
    rec, xv = orc.decode(dt, store[0][neuron[slots]]), orc.decode(dt, h)
    a = np.maximum(rec[:, :d] @ xv, 0) * (rec[:, d:2 * d] @ xv)
    assert np.max(np.abs(a)) < 2.0 ** 12 and np.max(np.abs(a) @ np.abs(rec[:, 2 * d:])) < 2.0 ** 6
    y = torch.zeros(d * W.ITEMSIZE[dt], dtype=torch.uint8, device=DEV)
    B.np_sparse_mlp(bufs.shape, 0, to_dev(h), to_dev(store[0][neuron]), to_dev(slots), n, y, bufs.ws)
    torch.cuda.synchronize()
    ref = orc.sparse_mlp(cfg, 0, h, store, neuron[slots])
    assert np.array_equal(decode_y(orc, dt, y.cpu().numpy()), decode_y(orc, dt, ref))
    assert B.np_device_error(bufs.ws) == 0


def chains_of_256(a, down):
    """sum_j a[j] down[j] in fp32 as 256 workgroups sum it row by row (one fused
    multiply-add a row), their sums met in the reduce kernel's order."""
    f32, F = np.float32, len(a)
    parts = np.zeros((256, down.shape[1]), f32)
    for j in range(F):  # workgroup b takes rows b, b + 256, ...; a[j] has 8 bits: the product is exact
        p = parts[j % 256]
        p[:] = (p.astype(np.float64) + np.float64(a[j]) * down[j]).astype(f32)
    v = parts.reshape(4, 4, 16, -1)  # row 64 h + 16 w + q: thread order within a column block
    acc = v[0].copy()
    for h in range(1, 4):
        acc += v[h]
    for bit in (1, 2, 4, 8):
        acc = acc + acc[:, np.arange(16) ^ bit]
    y = acc[0, 0].copy()
    for w in range(1, 4):
        y = y + acc[w, 0]
    return y.astype(np.float64)


@pytest.mark.parametrize("fused", ["0", "1"], ids=["two_kernels", "fused"])
@pytest.mark.parametrize("dense", [True, False], ids=["dense", "sparse"])
def test_mlp_fp32_sums_no_worse_than_256_chains(dense, fused, monkeypatch):
    """In fp32 the down projection of a long range is no further from the exact
    sum than 256 plain chains of rows would be, although fewer workgroups run:
    every g is 1 and every u has 8 bits, so the activations are exact and the
    sum's rounding is all there is.  6000 rows run on 188 workgroups of 32; the
    chains of 24 that 256 workgroups have are 1.16e-7 off, chains of 32 rows
    1.28e-7 (dense), sums by rounds of 4 that meet in fp64 0.75e-7."""
    d, F = 1024, 6000
    monkeypatch.setenv("NP_MLP_FUSED", fused)
    say(f"[mlp fp32 sums] dense {dense} fused {fused}")
    rng = np.random.default_rng(3)
    a = (rng.integers(1, 256, F) * rng.choice([-1, 1], F)).astype(np.float32) / 64
    rec = np.zeros((F, 3 * d), np.float32)
    rec[:, 0], rec[:, d] = 1.0, a
    rec[:, 2 * d:] = rng.standard_normal((F, d)).astype(np.float32)
    exact = a.astype(np.float64) @ rec[:, 2 * d:].astype(np.float64)
    x = torch.zeros(d, device=DEV)
    x[0] = 1.0
    y = torch.zeros(d, device=DEV)
    shape = B.make_shape(1, d, F, 8, F, F, "f32")
    ws = torch.zeros(B.np_workspace_size(shape), dtype=torch.uint8, device=DEV)
    res = torch.from_numpy(rec).to(DEV)
    if dense:
        B.np_dense_mlp(shape, res, x, y, ws)
    else:
        B.np_sparse_mlp(shape, 0, x, res, torch.arange(F, dtype=torch.int32, device=DEV), F, y, ws)
    torch.cuda.synchronize()
    err = np.linalg.norm(y.cpu().numpy() - exact)
    assert err <= np.linalg.norm(chains_of_256(a, rec[:, 2 * d:]) - exact)
    assert B.np_device_error(ws) == 0
