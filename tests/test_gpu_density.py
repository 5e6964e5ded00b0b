"""GPU parity of svoo_attention_density (offline profiling, attention density of Sec. 4.1) against
the fp64 oracle.  Prefix lengths are integers decided by floating point: a length must equal the
oracle's unless the oracle's cumulative sum passes tau by less than SLACK on one side of the
crossing (float32 logits and masses on the GPU against float64); then it may differ by a few."""
import math

import numpy as np
import pytest
import torch

from oracle import svoo_oracle as so
from paper_2603_18636_amd import svoo, synth
from tests import helpers as H

pytestmark = pytest.mark.gpu

SLACK = 2e-5        # float32 logits: relative error ~1e-6 on |s| ~ 10 -> masses good to ~1e-5


def compare_prefix(got, ref, max_near=None):
    diff = np.nonzero(got != ref["prefix_len"])[0]
    bad = diff[ref["slack"][diff] > SLACK]
    assert bad.size == 0, f"{bad.size} rows differ beyond rounding; first {bad[0]}: {got[bad[0]]} vs {ref['prefix_len'][bad[0]]}"
    if diff.size:
        rel = np.abs(got[diff] - ref["prefix_len"][diff]) / ref["prefix_len"][diff]
        assert (np.abs(got[diff] - ref["prefix_len"][diff]) <= 2 + 1e-3 * ref["prefix_len"][diff]).all(), rel.max()
    if max_near is not None:
        assert diff.size <= max_near
    return int(diff.size)


@pytest.mark.parametrize("dtype,d,grid,tau", [("bf16", 128, (6, 12, 20), 0.95), ("bf16", 64, (3, 3, 37), 0.5),
                                              ("f32", 64, (4, 16, 16), 0.95), ("f32", 128, (1, 3, 43), 0.9),
                                              ("bf16", 128, (1, 1, 64), 0.99), ("bf16", 64, (1, 1, 2), 0.95)])
def test_density_matches_oracle(dtype, d, grid, tau):
    cfg = synth.CONFIGS[1]
    heads = [synth.make_head(cfg, 2, hd, grid=grid, n_seeds=8, kq=1, kk=1, d=d, dtype=dtype) for hd in range(2)]
    q = np.stack([h["q"] for h in heads])
    k = np.stack([h["k"] for h in heads])
    n = q.shape[1]
    scale, tau32 = H.scale_of(d), float(np.float32(tau))
    plen, dens = svoo.attention_density(H.to_dev(q, dtype), H.to_dev(k, dtype), tau32, scale)
    plen, dens = H.to_np(plen), H.to_np(dens)
    for b in range(2):
        ref = so.attention_density(q[b], k[b], scale, tau32)
        near = compare_prefix(plen[b], ref, max_near=max(2, n // 100))
        assert abs(dens[b] - plen[b].mean() / n) < 1e-15
        if near == 0:     # same integers; only the order of the divisions differs
            assert abs(dens[b] - ref["density"]) <= 1e-14


@pytest.mark.parametrize("d,grid,copies", [(128, (6, 12, 20), 12), (128, (6, 12, 20), 24), (64, (3, 3, 37), 45),
                                           (64, (3, 3, 37), 90), (128, (1, 3, 43), 300)])
def test_density_in_every_launch_shape(d, grid, copies):
    """The rows of a workgroup are the fewest (32, 64 or 96) with which one round of 256 workgroups covers all rows,
    else 128; the small cases above all take 32.  Here two heads are repeated ``copies`` times so that the
    same data runs through workgroups of 128 rows and, with two heads, of 32 (n = 1440; n = 333, ragged last
    tile; n = 129, three 64-key tiles of which the last holds one key), each compared with the oracle, and
    every copy must equal the first.  64 and 96 rows: ``test_density_bracket_splits``."""
    cfg = synth.CONFIGS[1]
    heads = [synth.make_head(cfg, 7, hd, grid=grid, n_seeds=8, kq=1, kk=1, d=d, dtype="bf16") for hd in range(2)]
    q = np.tile(np.stack([h["q"] for h in heads]), (copies, 1, 1))
    k = np.tile(np.stack([h["k"] for h in heads]), (copies, 1, 1))
    n = q.shape[1]
    wgs = (n + 127) // 128 * 2 * copies
    assert wgs > 256
    scale, tau32 = H.scale_of(d), float(np.float32(0.95))
    plen, dens, passes = svoo.attention_density(H.to_dev(q, "bf16"), H.to_dev(k, "bf16"), tau32, scale, want_passes=True)
    plen, dens, passes = H.to_np(plen), H.to_np(dens), H.to_np(passes)
    for b in range(2):
        ref = so.attention_density(q[b], k[b], scale, tau32)
        compare_prefix(plen[b], ref, max_near=max(2, n // 100))
        assert (plen[b::2] == plen[b]).all() and (dens[b::2] == dens[b]).all() and (passes[b::2] == passes[b]).all()
    # 32-row workgroups on the same two heads
    plen4, _ = svoo.attention_density(H.to_dev(q[:2], "bf16"), H.to_dev(k[:2], "bf16"), tau32, scale)
    differ = int((H.to_np(plen4) != plen[:2]).sum())
    print(f"{wgs} workgroups: {differ} of {2 * n} prefix lengths differ from the launch of two heads")
    assert differ <= max(2, n // 100)


def test_density_row_subset_and_order():
    h = synth.make_head(synth.CONFIGS[1], 5, 0, grid=(6, 12, 20), n_seeds=8, kq=1, kk=1)
    q, k, n = h["q"][None], h["k"][None], h["q"].shape[0]
    rows = np.array([n - 1, 0, 17, 17, 700, 129], dtype=np.int32)        # any order, repeats allowed
    plen, dens = svoo.attention_density(H.to_dev(q, "bf16"), H.to_dev(k, "bf16"), 0.95, H.scale_of(128),
                                        rows=H.to_dev(rows))
    ref = so.attention_density(q[0], k[0], H.scale_of(128), float(np.float32(0.95)), rows=rows)
    compare_prefix(H.to_np(plen)[0], ref, max_near=0)
    assert abs(H.to_np(dens)[0] - ref["prefix_len"].mean() / n) <= 1e-14


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_density_single_key(dtype):
    x = synth.round_to_bf16(np.random.default_rng(0).standard_normal((3, 1, 128)).astype(np.float32))
    plen, dens = svoo.attention_density(H.to_dev(x, dtype), H.to_dev(x, dtype))       # default tau and scale
    assert (H.to_np(plen) == 1).all() and (H.to_np(dens) == 1.0).all()


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_density_ties_uniform_and_geometric(dtype):
    """Zero queries: every key ties, the prefix is ceil(tau n).  Keys -j ln2 / scale on one axis
    against a unit query: p_j ~ 2^-j, so the prefix for tau is ceil(log2(1 / (1 - tau)))."""
    n, d, scale = 200, 64, 0.25
    rng = np.random.default_rng(1)
    k = synth.round_to_bf16(rng.standard_normal((1, n, d)).astype(np.float32))
    q0 = np.zeros((1, n, d), dtype=np.float32)
    for tau in (0.95, 0.5, 1.0):
        plen, _ = svoo.attention_density(H.to_dev(q0, dtype), H.to_dev(k, dtype), tau, scale)
        assert (H.to_np(plen) == math.ceil(float(np.float32(tau)) * n)).all()
    # pairs of identical keys: ties inside the prefix are taken one at a time
    kd = np.repeat(k[:, : n // 2], 2, axis=1)
    qd = synth.round_to_bf16(rng.standard_normal((1, n, d)).astype(np.float32))
    plen, _ = svoo.attention_density(H.to_dev(qd, dtype), H.to_dev(kd, dtype), 0.9, scale)
    ref = so.attention_density(qd[0], kd[0], scale, float(np.float32(0.9)))
    compare_prefix(H.to_np(plen)[0], ref, max_near=2)
    kg = np.zeros((1, n, d), dtype=np.float32)
    kg[0, :, 0] = -np.arange(n) * 4.0                     # bf16-exact; scale ln2 / 4 makes p_j ~ 2^-j
    qg = np.zeros((1, n, d), dtype=np.float32)
    qg[0, :, 0] = 1.0
    sc = float(np.float32(math.log(2.0) / 4.0))
    for tau, want in ((0.9, 4), (0.6, 2), (0.99, 7)):
        plen, dens = svoo.attention_density(H.to_dev(qg, dtype), H.to_dev(kg, dtype), tau, sc)
        assert (H.to_np(plen) == want).all()
        assert abs(H.to_np(dens)[0] - want / n) < 1e-15


@pytest.mark.parametrize("dtype,d,n,n_rows,kind", [
    ("bf16", 128, 97, 33, "spread"), ("bf16", 64, 1000, 65, "ties"), ("bf16", 128, 4099, 97, "outlier"),
    ("bf16", 64, 8193, 129, "flat"), ("bf16", 128, 700, 700, "ties"), ("f32", 128, 1025, 31, "outlier"),
    ("f32", 64, 999, 70, "flat"), ("f32", 128, 3000, 65, "ties")])
def test_density_bracket_splits(dtype, d, n, n_rows, kind):
    """Row counts on both sides of 32, 64, 96 and 128 rows per workgroup (by repeating the head so that one
    round of the chip no longer holds them), and logits that the equal bins of the first histogram split
    badly: masses over hundreds of octaves, a few values with more ties than a list holds, one key far
    above the rest, keys within a few float steps of each other.  Checked against the oracle; a cumulative
    mass within SLACK of tau may decide either way (float32 logits: the derivation above)."""
    rng = np.random.default_rng(n)
    q = rng.standard_normal((1, n, d)).astype(np.float32)
    k = rng.standard_normal((1, n, d)).astype(np.float32)
    if kind == "spread":
        k *= 40.0
    elif kind == "ties":
        k = k[:, rng.integers(0, 7, n)]
    elif kind == "outlier":
        k[0, n // 2] = 50.0 * q[0, 0]
    else:
        k = 1.0 + np.round(2.0 * k) / 128.0
    if dtype == "bf16":
        q, k = synth.round_to_bf16(q), synth.round_to_bf16(k)
    rows = rng.integers(0, n, n_rows).astype(np.int32)
    rows[0] = 0
    tau32 = float(np.float32(0.95))
    ref = so.attention_density(q[0], k[0], H.scale_of(d), tau32, rows=rows)
    for copies in (1, 9, 120):
        plen, _ = svoo.attention_density(H.to_dev(np.tile(q, (copies, 1, 1)), dtype), H.to_dev(np.tile(k, (copies, 1, 1)), dtype),
                                         tau32, H.scale_of(d), rows=H.to_dev(rows))
        plen = H.to_np(plen)
        compare_prefix(plen[0], ref, max_near=max(2, n_rows // 20))
        assert (plen == plen[0]).all()


def test_density_full_size_head_of_config2():
    """One head at the real shape (75,600 keys), 1,024 sampled query rows, tau = 0.95."""
    cfg = synth.CONFIGS[2]
    h = synth.make_head(cfg, 0, 2)
    rows = np.sort(np.random.default_rng(3).choice(cfg.n, 1024, replace=False)).astype(np.int32)
    scale = H.scale_of(cfg.d)
    plen, dens, passes = svoo.attention_density(H.to_dev(h["q"][None], "bf16"), H.to_dev(h["k"][None], "bf16"), 0.95,
                                                scale, rows=H.to_dev(rows), want_passes=True)
    torch.cuda.synchronize()
    assert 3 <= int(H.to_np(passes)[0]) <= 40
    ref = so.attention_density(h["q"], h["k"], scale, float(np.float32(0.95)), rows=rows, chunk=256)
    plen = H.to_np(plen)[0]
    near = compare_prefix(plen, ref)
    d_gpu, d_ref = H.to_np(dens)[0], ref["density"]
    print(f"config 2 density: gpu {d_gpu:.6f} oracle {d_ref:.6f}, {near} of 1024 prefix lengths differ within rounding")
    assert abs(d_gpu - d_ref) <= 1e-4 * d_ref


@pytest.mark.parametrize("dtype,d,n", [("bf16", 128, 97), ("bf16", 64, 1000), ("f32", 128, 333), ("f32", 64, 64)])
def test_density_with_logits_that_are_no_finite_numbers(dtype, d, n):
    """Products beyond float32's range and keys or queries that hold a NaN.  A row with an infinite logit has the number
    of its logits above -inf as its length, a key whose logit is NaN weighs nothing, a row of NaNs has length 1;
    the other rows of the workgroup are the oracle's."""
    rng = np.random.default_rng(n)
    q, k = (rng.standard_normal((1, n, d)).astype(np.float32) for _ in range(2))
    q[0, :, 0] = 0.0
    q[0, 3::5, 0] = 2.0 ** 100
    q[0, 4::5, 0] = -(2.0 ** 100)
    k[0, :, 0] = 0.0
    low = rng.choice(n, 7, replace=False)
    k[0, low, 0] = -(2.0 ** 100)
    q[0, 2] = np.nan
    lost = int(rng.integers(n))
    k[0, lost, d - 1] = np.nan
    if dtype == "bf16":
        q, k = synth.round_to_bf16(q), synth.round_to_bf16(k)
    tau32 = float(np.float32(0.95))
    got = {}
    for bad in (False, True):               # without and with the key that is NaN
        kk = k if bad else np.nan_to_num(k)
        plen, _ = svoo.attention_density(H.to_dev(q, dtype), H.to_dev(kk, dtype), tau32, H.scale_of(d))
        got[bad] = H.to_np(plen)[0]
        keys = np.arange(n) != lost if bad else np.ones(n, dtype=bool)
        left = int(keys.sum())
        row = np.arange(n)
        assert got[bad][2] == 1
        assert (got[bad][(row % 5 == 3) & (row != 2)] == left - int(keys[low].sum())).all()      # -inf logits
        assert (got[bad][row % 5 == 4] == left).all()                                            # +inf logits
        rows = row[(row % 5 < 3) & (row != 2)]
        ref = so.attention_density(q[0], kk[0][keys], H.scale_of(d), tau32, rows=rows)
        compare_prefix(got[bad][rows], ref, max_near=max(2, n // 50))


@pytest.mark.parametrize("dtype,d,n,rows", [("bf16", 128, 97, 97), ("bf16", 64, 1000, 300), ("f32", 128, 333, 65), ("f32", 64, 1, 1)])
def test_density_of_rows_with_equal_logits_takes_one_pass(dtype, d, n, rows):
    """Zero queries (padding): the length is known once the extremes are, also in a workgroup of other rows."""
    rng = np.random.default_rng(n)
    q, k = (synth.round_to_bf16(rng.standard_normal((1, n, d)).astype(np.float32)) for _ in range(2))
    index = H.to_dev(rng.choice(n, rows, replace=False).astype(np.int32))
    for tau in (0.3, 0.95, 1.0):
        tau32 = float(np.float32(tau))
        plen, _, passes = svoo.attention_density(H.to_dev(0.0 * q, dtype), H.to_dev(k, dtype), tau, H.scale_of(d), rows=index,
                                                 want_passes=True)
        assert (H.to_np(plen) == math.ceil(tau32 * n)).all() and (H.to_np(passes) == 1).all()
        half = q.copy()
        half[0, ::2] = 0.0
        plen, _ = svoo.attention_density(H.to_dev(half, dtype), H.to_dev(k, dtype), tau, H.scale_of(d), rows=index)
        even = H.to_np(index) % 2 == 0
        assert (H.to_np(plen)[0][even] == math.ceil(tau32 * n)).all()
        if tau < 1.0:
            ref = so.attention_density(half[0], k[0], H.scale_of(d), tau32, rows=H.to_np(index))
            compare_prefix(H.to_np(plen)[0], ref, max_near=max(2, rows // 50))


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_density_sees_the_mass_of_a_million_tiny_keys(dtype):
    """One key of mass 1 and 2^20 - 1 of mass 2^-43, together 2^-23 more: a share 1 - 2^-24 of it needs the large
    one and half of the others.  Nothing in units of 2^-41, in which 2^20 keys of mass 1 are summed up.  Bound:
    scale and logit are rounded to 2^-24 each, which moves the exponent 43 by 5e-6 at most."""
    n, d = 1 << 20, 64
    q = torch.zeros((1, n, d), dtype=H.torch_dtype(dtype), device=H.DEV)
    k = torch.zeros_like(q)
    q[0, :, 0] = 1.0
    k[0, :, 0] = -1.0
    k[0, 7, 0] = 0.0
    rows = torch.arange(40, dtype=torch.int32, device=H.DEV)
    plen, _ = svoo.attention_density(q, k, float(np.float32(1.0 - 2.0 ** -24)), 43.0 * math.log(2.0), rows=rows)
    assert (np.abs(H.to_np(plen) - 2.0 ** 19) <= 16).all()


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16", 64), ("f32", 128), ("f32", 64)])
@pytest.mark.parametrize("group", [1, 4, 5, 32, 5003])
def test_density_does_not_hang_on_the_order_of_the_keys(dtype, d, group):
    """Runs of ``group`` keys of neighbouring logits: from none to all 16 of a lane's logits lie inside the bracket, on
    both sides of the rule that picks a few one by one.  Masses are integers, so the lengths equal those of the
    unordered keys."""
    rng = np.random.default_rng(d)
    n = 5003
    head = synth.make_head(synth.CONFIGS[1], 4, 0, grid=(1, 1, n), n_seeds=8, kq=1, kk=1, d=d, dtype=dtype)
    q, k = head["q"][:97], head["k"]
    by_logit = np.argsort(k.astype(np.float64) @ q[0].astype(np.float64))
    runs = [by_logit[i:i + group] for i in range(0, n, group)]
    order = np.concatenate([runs[i] for i in rng.permutation(len(runs))])
    rows = np.zeros((n, d), q.dtype)
    rows[:97] = q[0] + 1e-3 * (q - q[0])             # rows that order the keys much as row 0 does
    rows = H.to_np(H.to_dev(rows, dtype).float()).astype(q.dtype)
    scale, tau = H.scale_of(d), float(np.float32(0.95))
    which = H.to_dev(np.arange(97, dtype=np.int32))
    got = [H.to_np(svoo.attention_density(H.to_dev(rows[None], dtype), H.to_dev(np.ascontiguousarray(x)[None], dtype), tau, scale,
                                          rows=which)[0])[0] for x in (k, k[order])]
    assert (got[0] == got[1]).all()
    ref = so.attention_density(rows[:97], k, scale, tau)
    compare_prefix(got[1], ref)
