"""GPU parity of the independent k-means partitioner (ablation "w/o On") and of the attention-recall
diagnostic built on the kernels' log-sum-exp outputs, against the fp64 oracle."""
import math

import numpy as np
import pytest
import torch

from oracle import svoo_oracle as so
from paper_2603_18636_amd import svoo, synth
from tests import helpers as H

pytestmark = pytest.mark.gpu


def small_head(layer=0, head=0, grid=(6, 12, 20), n_seeds=24, kq=24, kk=20, d=128, dtype="bf16"):
    return synth.make_head(synth.CONFIGS[1], layer, head, grid=grid, n_seeds=n_seeds, kq=kq, kk=kk, d=d, dtype=dtype)


def run_and_check(xd, x, init_idx, iters, b=0, what="k-means"):
    """svoo_kmeans on device tensor xd [bh, n, d] next to the oracle on slice b, iteration by iteration:
    a label difference must be a proven near-tie of that iteration, after which the oracle follows the
    GPU, so counts and centroids are always compared.  Returns the number of near-tie differences."""
    steps, _ = H.gpu_kmeans_steps(xd, H.to_dev(init_idx), iters)
    out = svoo.kmeans(xd, H.to_dev(init_idx), iters, want_inertia=True)
    assert (H.to_np(out["labels"]) == steps[iters - 1]).all()
    ref = H.resync_kmeans(x, init_idx[b], iters, H.slice_steps(steps, b), what=what)
    assert (H.to_np(out["labels"])[b] == ref["labels"]).all()
    assert (H.to_np(out["counts"])[b] == ref["counts"]).all()
    np.testing.assert_array_equal(H.to_np(out["c"])[b], ref["c"].astype(np.float32))
    inertia = H.to_np(out["inertia"])[b]
    for it, j_ref in enumerate(ref["inertia"]):
        if j_ref is None or sum(ref["near_steps"][:it]) > 0:
            continue              # a moved label changes the sums from there on
        np.testing.assert_allclose(inertia[it], j_ref, rtol=1e-9)
    return ref["near"]


@pytest.mark.parametrize("dtype,d,iters", [("bf16", 128, 3), ("f32", 64, 5), ("bf16", 64, 2), ("f32", 128, 1)])
def test_kmeans_matches_oracle(dtype, d, iters):
    h = small_head(d=d, dtype=dtype)
    for side, idx in (("k", "init_k_idx"), ("q", "init_q_idx")):
        x = h[side]
        run_and_check(H.to_dev(x[None], dtype), x, h[idx][None], iters)


def test_kmeans_heads_are_independent_and_k_1024():
    """Three heads in one call; 1024 clusters on 5000 tokens (32-centroid blocks, many near-empty)."""
    cfg = synth.CONFIGS[1]
    heads = [synth.make_head(cfg, 0, hd, grid=(5, 25, 40), n_seeds=64, kq=1024, kk=1000) for hd in range(3)]
    x = np.stack([h["k"] for h in heads])
    for name, k in (("init_q_idx", 1024), ("init_k_idx", 1000)):
        idx = np.stack([h[name] for h in heads])
        for b in range(3):
            run_and_check(H.to_dev(x, "bf16"), x[b], idx, 2, b)


def test_kmeans_warm_start_duplicates_and_far_centroid():
    h = small_head(dtype="bf16")
    k = h["k"]
    c0 = k[h["init_k_idx"]].astype(np.float32)
    c0[5] = c0[2]                      # duplicate: ties go to the lower index, cluster 5 stays empty
    c0[7] = 300.0                      # far from every token: empty, must keep its centroid
    for iters in (1, 2):   # after the first update cluster 2 has moved and cluster 5 may win tokens
        out = svoo.kmeans(H.to_dev(k[None], "bf16"), None, iters, init_c=H.to_dev(c0[None]))
        ref = so.kmeans(k, None, iters, init_c=c0)
        assert (H.to_np(out["labels"])[0] == ref["labels"]).all()
        counts = H.to_np(out["counts"])[0]
        assert counts[7] == 0 and (counts == ref["counts"]).all()
        got_c = H.to_np(out["c"])[0]
        assert (got_c[7] == 300.0).all()
        if iters == 1:
            assert counts[5] == 0 and (got_c[5] == c0[2]).all()
        np.testing.assert_array_equal(got_c, ref["c"].astype(np.float32))


def test_kmeans_full_size_head_of_config2():
    """One head at the real shape (75,600 tokens, 256 clusters, d = 128), two iterations."""
    cfg = synth.CONFIGS[2]
    h = synth.make_head(cfg, 0, 1)
    for side, idx in (("q", "init_q_idx"), ("k", "init_k_idx")):
        near = run_and_check(H.to_dev(h[side][None], "bf16"), h[side], h[idx][None], 2,
                             what=f"configs[2] k-means({side})")
        print(f"config 2 k-means({side}): {near} near-tie label differences of {cfg.n}")


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("f32", 64)])
def test_layer_with_kmeans_partitioner_and_recall(dtype, d):
    """Whole path with the independent partitioner, then the recall diagnostic from the two
    log-sum-exp outputs against the oracle's dense-softmax definition."""
    h = small_head(d=d, dtype=dtype, layer=3)
    q, k, v = h["q"], h["k"], h["v"]
    kq, kk, iters, keep = 24, 20, 2, 0.3
    scale = H.scale_of(d)
    dev = {n: H.to_dev(h[n][None], dtype) for n in "qkv"}
    layer = svoo.Layer(1, q.shape[0], d, H.torch_dtype(dtype), kq, kk, H.DEV)
    keep_dev = H.to_dev(np.array([keep], dtype=np.float32))
    out = layer.run(dev["q"], dev["k"], dev["v"], H.to_dev(h["init_q_idx"][None]), H.to_dev(h["init_k_idx"][None]),
                    iters, keep_dev, 1.0, 0.0, scale, partitioner="kmeans")
    ref = so.layer(q, k, v, h["init_q_idx"], h["init_k_idx"], iters, float(np.float32(keep)), 1.0, 0.0, scale,
                   partitioner="kmeans")
    assert (H.to_np(layer.labels_q)[0] == ref["labels_q"]).all()
    assert (H.to_np(layer.labels_k)[0] == ref["labels_k"]).all()
    assert (H.to_np(layer.bitmap)[0].astype(bool) == ref["mask"]).all()
    H.assert_attn_close(H.to_np(out)[0], ref["out"], dtype, "k-means layer")
    rec = H.to_np(layer.row_recall(dev["q"], dev["k"], dev["v"], scale))[0]
    rec_ref = so.row_recall(q, k, ref["labels_q"], ref["labels_k"], ref["mask"], scale, np.arange(q.shape[0]))
    tol = 3e-2 if dtype == "bf16" else 1e-4
    assert np.abs(rec - rec_ref).max() <= tol
    assert abs(rec.mean() - rec_ref.mean()) <= tol / 5
    assert 0.0 < rec_ref.mean() < 1.0


@pytest.mark.parametrize("dtype,d,n", [("bf16", 128, 700), ("bf16", 64, 257), ("f32", 128, 300), ("f32", 64, 513)])
@pytest.mark.parametrize("tie", [False, True])
def test_kmeans_zero_and_tiny_tokens(dtype, d, n, tie):
    """A zero token's scores hang on the centroids alone: the pre-filter may decide it, unless the two shortest
    centroids are equally long (the lower index wins then).  Tokens of 1e-25 are the same to float32."""
    rng = np.random.default_rng(n)
    c = (2.0 + rng.random((37, d))).astype(np.float32) * rng.choice([-1.0, 1.0], (37, d)).astype(np.float32)
    c[5] = synth.round_to_bf16(0.5 * c[5])
    c[3] = -c[5] if tie else c[3]
    x = rng.standard_normal((n, d)).astype(np.float32)
    x[n - 120:] = 0.0
    x[10:20] *= 1e-25
    if dtype == "bf16":
        x = synth.round_to_bf16(x)
    out = svoo.kmeans(H.to_dev(x[None], dtype), iters=1, init_c=H.to_dev(c[None]))
    labels = H.to_np(out["labels"])[0]
    ref = so.kmeans(x, None, 1, init_c=c)
    H.compare_labels(labels, ref["labels"], ref["trace"][0]["best"], ref["trace"][0]["second"])
    assert (labels[n - 120:] == (3 if tie else 5)).all()


@pytest.mark.parametrize("dtype,d,n", [("bf16", 128, 259), ("f32", 128, 515), ("f32", 64, 300), ("bf16", 64, 266)])
def test_a_centroid_that_is_nan_wins_no_token(dtype, d, n):
    """One own-side centroid is NaN (what a NaN token leaves behind): the other tokens go to the best of the other
    centroids, decided in float64 in workgroups with 256 and with a few open tokens, on all three paths."""
    rng = np.random.default_rng(n)
    x = rng.standard_normal((n, d)).astype(np.float32)
    x = synth.round_to_bf16(x) if dtype == "bf16" else x
    for k in (24, 90):
        c = rng.standard_normal((k, d)).astype(np.float32)
        for lost in (0, 7, k - 1):
            bad = c.copy()
            bad[lost, d // 2] = np.nan
            rest = np.delete(np.arange(k), lost)
            got = H.to_np(svoo.kmeans(H.to_dev(x[None], dtype), iters=1, init_c=H.to_dev(bad[None]))["labels"])[0]
            ref = so.kmeans(x, None, 1, init_c=c[rest])
            assert (got != lost).all()
            H.compare_labels(got - (got > lost), ref["labels"], ref["trace"][0]["best"], ref["trace"][0]["second"])
            opp = rng.standard_normal((20, d)).astype(np.float32)
            ref = H.oracle_assign(x, c[rest], opp)
            got = H.to_np(svoo.assign(H.to_dev(x[None], dtype), H.to_dev(bad[None]), H.to_dev(opp[None])))[0]
            assert (got != lost).all()
            H.compare_labels(got - (got > lost), *ref)
            q = H.to_dev(rng.standard_normal((1, n, d)).astype(np.float32), dtype)
            got = H.to_np(svoo.cocluster(q, H.to_dev(x[None], dtype), iters=1, init_cq=H.to_dev(opp[None]),
                                         init_ck=H.to_dev(bad[None]))["labels_k"])[0]
            H.compare_labels(got - (got > lost), *ref)


def split_worst_rows(rng, n, d):
    """Rows whose elements split worst into two bf16 terms: half-way between two bf16 numbers next to a power of two
    (lower terms of either sign, 2^-8 of the element), with a remainder behind the lower term."""
    x = rng.choice([1 + 2.0 ** -8, 1 + 3 * 2.0 ** -8], (n, d)) - rng.choice([0.0, 2.0 ** -17, 2.0 ** -16 + 2.0 ** -17], (n, d))
    return x * rng.choice([-1.0, 1.0], (n, d)) * 2.0 ** rng.integers(-1, 2, (n, d))


@pytest.mark.parametrize("d,n,k", [(64, 700, 40), (128, 700, 33), (128, 9000, 130)])
@pytest.mark.parametrize("scale", [1.0, 1e-17, 1e17, 3e18])
@pytest.mark.parametrize("worst", [False, True])
def test_float32_labels_with_centroids_closer_than_two_bf16_terms_tell(d, n, k, scale, worst):
    """Float32 tokens and centroids in pairs 2^-14 .. 2^-22 apart: the pre-filter on two bf16 terms of each must leave
    open what it cannot tell, down to products that are subnormal, up to squares near the end of float32 and beyond."""
    rng = np.random.default_rng(d + n)
    scale = 2.0 ** round(np.log2(scale)) if worst else scale
    x = (scale * (split_worst_rows(rng, n, d) if worst else rng.standard_normal((n, d))))[None].astype(np.float32)
    c = x[:, rng.choice(n, k, replace=False)].copy()
    for j in range(1, k, 2):
        c[0, j] = c[0, j - 1] * np.float32(1 + 2.0 ** -(14 + j % 9))
    got = H.to_np(svoo.kmeans(H.to_dev(x, "f32"), iters=1, init_c=torch.from_numpy(c).to(H.DEV))["labels"])[0]
    xx, cc = x[0].astype(np.float64) / scale, c[0].astype(np.float64) / scale
    score = 2.0 * xx @ cc.T - (cc * cc).sum(1)
    best = score.argmax(1)
    gap = score[np.arange(n), best] - score[np.arange(n), got]
    assert (gap <= 1e-13 * np.abs(score).max()).all(), (int((gap > 0).sum()), float(gap.max()))


@pytest.mark.parametrize("d,n,k", [(64, 700, 40), (128, 700, 32), (64, 9000, 40), (128, 9000, 130)])
@pytest.mark.parametrize("scale", [1.0, 2.0 ** 57, 2.0 ** 60, 2.0 ** 62])
@pytest.mark.parametrize("worst", [False, True])
def test_float32_co_clustering_with_anchors_closer_than_two_bf16_terms_tell(d, n, k, scale, worst):
    """The same for co-clustering, on the path of few clusters and tokens and on the general one: own-side centroids in
    pairs that differ by 2^-14 .. 2^-22 element-wise, scores <x, W_j> in float64 beside the labels."""
    rng = np.random.default_rng(d + n + k)
    rows = (lambda m: split_worst_rows(rng, m, d)) if worst else (lambda m: rng.standard_normal((m, d)))
    x, q, opp = ((scale * rows(m)).astype(np.float32) for m in (n, n, 24))
    own = x[rng.choice(n, k, replace=False)].copy()
    for j in range(1, k, 2):
        own[j] = own[j - 1] * (1 + 2.0 ** -(14 + j % 9) * rng.uniform(-1, 1, d)).astype(np.float32)
    got = H.to_np(svoo.cocluster(H.to_dev(q[None], "f32"), H.to_dev(x[None], "f32"), iters=1, init_cq=H.to_dev(opp[None]),
                                 init_ck=H.to_dev(own[None]))["labels_k"])[0]
    xx, oo, pp = (a.astype(np.float64) / scale for a in (x, own, opp))
    aff = oo @ pp.T
    score = (xx @ pp.T) @ (aff / np.linalg.norm(aff, axis=1, keepdims=True)).T
    gap = score.max(1) - score[np.arange(n), got]
    assert (gap <= 1e-12 * np.abs(score).max()).all(), (int((gap > 0).sum()), float(gap.max()))


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("partitioner", ["kmeans", "cocluster"])
def test_large_tokens_take_no_longer(dtype, partitioner):
    """Scores between 1e37 and the end of float32 go through the pre-filter like any others: a power of two changes
    neither a label nor the time (deciding every token in float64 takes twice as long)."""
    gen = torch.Generator(device=H.DEV).manual_seed(7)
    x, y = (torch.randn(4, 30000, 128, generator=gen, device=H.DEV).to(H.torch_dtype(dtype)) for _ in range(2))
    labels, times = [], []
    for scale in (1.0, 2.0 ** 59):
        xs, ys = x * scale, y * scale
        cx, cy = xs[:, :160].float().contiguous(), ys[:, :160].float().contiguous()
        run = (lambda: svoo.kmeans(xs, iters=1, init_c=cx)["labels"]) if partitioner == "kmeans" else \
            (lambda: svoo.cocluster(xs, ys, iters=1, init_cq=cx, init_ck=cy)["labels_k"])
        labels.append(run())
        took = []
        for _ in range(20):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            run()
            b.record()
            b.synchronize()
            took.append(a.elapsed_time(b))
        times.append(min(took))
    assert torch.equal(*labels)
    assert times[1] < 1.25 * times[0], times


@pytest.mark.parametrize("dtype,d,n", [("bf16", 128, 700), ("f32", 128, 700), ("bf16", 64, 9000), ("f32", 64, 9000)])
@pytest.mark.parametrize("tiny", [2.0 ** -30, 2.0 ** -40])
def test_anchors_whose_scores_no_float32_holds(dtype, d, n, tiny):
    """Rows of the score matrix beyond float32 (elements, or only their norms) against tokens so small that their scores
    are ordinary numbers: no bound in float32 covers them, so every token is decided in float64."""
    rng = np.random.default_rng(d)
    bits = lambda a: synth.round_to_bf16(a.astype(np.float32))
    x, own = bits(tiny * rng.standard_normal((n, d))), bits(tiny * rng.standard_normal((30, d)))
    opp = bits(2.0 ** 126 * rng.uniform(1.0, 1.9, (24, d)) * rng.choice([-1.0, 1.0], (24, d)))
    own[7] = 2.0 ** -24 * own[7] + 0.5 * own[8]
    got = H.to_np(svoo.assign(H.to_dev(x[None], dtype), H.to_dev(own[None]), H.to_dev(opp[None])))[0]
    both = H.to_np(svoo.cocluster(H.to_dev(x[None], dtype), H.to_dev(x[None], dtype), iters=1, init_cq=H.to_dev(opp[None]),
                                  init_ck=H.to_dev(own[None]))["labels_k"])[0]
    xx, oo, pp = x.astype(np.float64), own.astype(np.float64), opp.astype(np.float64) / 2.0 ** 126
    aff = oo @ pp.T
    score = (xx @ pp.T) @ (aff / np.linalg.norm(aff, axis=1, keepdims=True)).T
    for labels in (got, both):
        gap = score.max(1) - score[np.arange(n), labels]
        assert (gap <= 1e-12 * np.abs(score).max()).all(), (int((gap > 0).sum()), float(gap.max() / np.abs(score).max()))


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16", 64), ("f32", 128), ("f32", 64)])
@pytest.mark.parametrize("k", [1, 2, 17, 31, 32, 33, 63, 65, 97, 1000])
@pytest.mark.parametrize("twins", [False, True])
def test_every_place_of_a_block_of_centroids_can_win(dtype, d, k, twins):
    """One token per centroid, on it: its label is that centroid, at every place of the 32-centroid blocks and in
    short last blocks.  Twins: centroids 2i and 2i + 1 coincide (a tie inside one pair of scores), the lower wins."""
    rng = np.random.default_rng(k)
    x = rng.standard_normal((k, d)).astype(np.float32)
    want = np.arange(k)
    if twins:
        x[1::2] = x[:k - 1:2] if k % 2 else x[::2]
        want[1::2] -= 1
    order = rng.permutation(k)                     # token order[j] is centroid j
    tokens = np.empty_like(x)
    tokens[order] = x
    xd = H.to_dev(tokens[None], dtype)
    out = svoo.kmeans(xd, H.to_dev(order[None].astype(np.int32)), 1)
    assert (H.to_np(out["labels"])[0][order] == want).all()
