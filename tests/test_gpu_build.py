"""Index construction on the MI355X against the oracle (Section 4.1), bit for bit:
centroids after k-means, assignment, offsets, document ids, packed codes, bucket
cutoffs and weights; then a search over the device-built index."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
import synth

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)


def _inputs(seed, n_docs, max_len, n_c=64):
    wl = synth.random_small_workload(seed, n_centroids=n_c, n_docs=n_docs, max_len=max_len, nbits=4)
    data = synth.make_index(wl, with_queries=True, workers=1)
    lens = data.doc_lengths.astype(np.int64)
    X = synth.token_vectors(data.workload, np.arange(int(lens.sum())))
    docs = np.repeat(np.arange(len(lens)), lens).astype(np.int32)
    return data, X, docs, lens


def _build_both(X, docs, n_docs, C0, sample, iterations, nbits, n_quant, label):
    import torch

    import paper_2501_17788_amd as w

    say(f"[{label}] n={len(X)} n_c={len(C0)} sample={len(sample)} it={iterations} b={nbits} n_quant={n_quant}")
    got = w.build_index(torch.from_numpy(X).cuda(), torch.from_numpy(docs).cuda(), n_docs, C0, sample,
                        iterations, nbits, n_quant)
    got = {k: v.cpu().numpy() for k, v in got.items()}
    want = oracle.build_index(X, docs, C0, sample, iterations, nbits, n_quant)
    for key in ("assign", "centroids", "offsets", "doc_ids", "codes", "cutoffs", "weights"):
        assert np.array_equal(got[key], want[key]), f"{label}: {key} differs"
    return got, want


@pytest.mark.parametrize("nbits", [1, 2, 4, 8])
def test_build_matches_oracle(nbits):
    import paper_2501_17788_amd as w

    data, X, docs, lens = _inputs(30 + nbits, n_docs=600, max_len=40, n_c=128)
    sample = w.sample_passages(lens, c=12.0, seed=nbits)
    C0 = w.initial_centroids(X, sample, 128, seed=nbits)
    _build_both(X, docs, len(lens), C0, sample, 4, nbits, 1500, label=f"b={nbits}")


def test_build_many_tiles_and_radix_passes():
    """600 centroids (two 8-bit passes of the stable sort by cluster) over about 60k tokens
    (15 tiles of 4,096 keys), quantiles over 20,000 tokens (2.56M residual components: four
    passes over 625 tiles): the hand-written sorts and prefix sums at several tiles."""
    import paper_2501_17788_amd as w

    data, X, docs, lens = _inputs(44, n_docs=3000, max_len=40, n_c=600)
    sample = w.sample_passages(lens, c=20.0, seed=5)
    C0 = w.initial_centroids(X, sample, 600, seed=6)
    assert len(X) > 8 * 4096
    _build_both(X, docs, len(lens), C0, sample, 2, 2, 20000, label="600 centroids, 20k quantile tokens")


def test_build_edge_cases():
    import paper_2501_17788_amd as w

    data, X, docs, lens = _inputs(40, n_docs=200, max_len=12, n_c=48)
    sample = w.sample_passages(lens, c=5.0, seed=1)
    C0 = w.initial_centroids(X, sample, 48, seed=2)
    _build_both(X, docs, len(lens), C0, sample, 0, 4, len(X), label="no k-means step, all tokens for quantiles")
    _build_both(X, docs, len(lens), C0[:1], sample[:1], 3, 2, 1, label="one centroid, one sample token")
    C1 = C0.copy()
    C1[7] = C1[3]  # duplicate centroids: ties go to the lower id
    C1[20] = C1[3]
    got, _ = _build_both(X, docs, len(lens), C1, sample, 2, 4, 200, label="duplicate centroids")


@pytest.mark.parametrize("n_c", [1, 127, 129, 256, 257, 640])
def test_build_nearest_centroid_blocks(n_c):
    """The nearest-centroid search works on tiles of 128 centroids and keeps two tiles per lane:
    centroid counts around a tile's edge, and sets in which every third centroid coincides, so that
    more tiles tie than a lane keeps (every centroid is then scored; ties go to the lowest id), which
    up to two tiles cannot."""
    import paper_2501_17788_amd as w

    data, X, docs, lens = _inputs(60, n_docs=500, max_len=40, n_c=64)
    sample = w.sample_passages(lens, c=30.0, seed=1)
    C0 = w.initial_centroids(X, sample, n_c, seed=2)
    _build_both(X, docs, len(lens), C0, sample, 1, 4, 300, label=f"{n_c} centroids")
    C0[1::3] = C0[0]
    _build_both(X, docs, len(lens), C0, sample, 1, 2, 300, label=f"{n_c} centroids, a third of them equal")


@pytest.mark.parametrize("extra", [1, 70001])
def test_build_second_chunk_of_tokens(extra):
    """Tokens are assigned 2^19 at a time: one split of the centroids in a whole chunk, several in a
    smaller last one, with tokens of coinciding centroids in both."""
    n, n_c = (1 << 19) + extra, 500
    rng = np.random.default_rng(extra)
    C = rng.standard_normal((n_c, 128), dtype=np.float32)
    C[7::20] = C[7]
    C /= np.linalg.norm(C, axis=1, keepdims=True)
    X = C[rng.integers(0, n_c, n)] + 0.1 * rng.standard_normal((n, 128), dtype=np.float32)
    X /= np.linalg.norm(X, axis=1, keepdims=True)
    docs = (np.arange(n) // 50).astype(np.int32)
    _build_both(X, docs, int(docs[-1]) + 1, C, np.arange(0, n, 1000, dtype=np.int64), 1, 2, 1000, label="2^19 tokens and more")


@pytest.mark.parametrize("same,spread", [(30, 0.0), (130, 1e-4), (700, 0.0), (2500, 3e-4), (4500, 6e-4)])
def test_build_close_centroids(same, spread):
    """Tokens with more centroids near their best than the product keeps tiles for, a number of them
    that is no multiple of the 16 that share a workgroup: lists of coinciding and of close centroids
    per token, and more than the 2,048 that a list holds."""
    import paper_2501_17788_amd as w

    data, X, docs, lens = _inputs(62, n_docs=400, max_len=30, n_c=64)
    rng = np.random.default_rng(same)
    n_c = same + 77
    C = rng.standard_normal((n_c, 128)).astype(np.float32)
    C /= np.linalg.norm(C, axis=1, keepdims=True)
    where = rng.permutation(n_c)[:same]
    C[where] = C[where[0]] + spread * rng.standard_normal((same, 128)).astype(np.float32)
    near = rng.permutation(len(X))[:777]
    X = X.copy()
    X[near] = C[where[0]] + 0.1 * rng.standard_normal((len(near), 128)).astype(np.float32)
    X[near] /= np.linalg.norm(X[near], axis=1, keepdims=True)
    _build_both(X, docs, len(lens), C, np.sort(near[:500]).astype(np.int64), 1, 4, 300, label=f"{same} centroids within {spread}")


def test_build_refuses_too_many_equal_centroids():
    """Centroids equal to a token's best are accepted up to 1,024; more are WARP_ENOTSUP."""
    import torch

    import paper_2501_17788_amd as w

    data, X, docs, lens = _inputs(61, n_docs=200, max_len=20, n_c=64)
    sample = np.arange(64, dtype=np.int64)
    for n_equal in (1000, 1100):
        C = np.repeat(X[:1], n_equal + 8, axis=0)
        C[n_equal:] = X[100:108]
        say(f"[{n_equal} equal centroids]")
        if n_equal <= 1024:
            _build_both(X[:300], docs[:300], len(lens), C, sample, 0, 4, 100, label=f"{n_equal} equal centroids")
            continue
        with pytest.raises(w.WarpError) as e:
            w.build_index(torch.from_numpy(X[:300]).cuda(), torch.from_numpy(docs[:300]).cuda(), len(lens), C, sample, 0, 4,
                          100)
        assert e.value.code == w.ENOTSUP


def test_build_errors():
    import torch

    import paper_2501_17788_amd as w

    data, X, docs, lens = _inputs(41, n_docs=50, max_len=6, n_c=16)
    sample = w.sample_passages(lens, c=5.0, seed=1)
    C0 = w.initial_centroids(X, sample, 16, seed=2)
    Xt, Dt = torch.from_numpy(X).cuda(), torch.from_numpy(docs).cuda()
    Z = C0.copy()
    Z[2] = 0
    with pytest.raises(w.WarpError) as e:
        w.build_index(Xt, Dt, len(lens), Z, sample, 1, 4, 10)
    assert e.value.code == w.EINVAL and "zero" in e.value.msg
    bad = sample.copy()
    bad[0] = len(X)
    with pytest.raises(w.WarpError) as e:
        w.build_index(Xt, Dt, len(lens), C0, bad, 1, 4, 10)
    assert e.value.code == w.EINVAL and "sample id" in e.value.msg
    with pytest.raises(w.WarpError) as e:
        w.build_index(Xt * 1.5, Dt, len(lens), C0, sample, 1, 4, 10)
    assert e.value.code == w.EINVAL and "norm" in e.value.msg
    with pytest.raises(w.WarpError) as e:
        w.build_index(Xt, Dt, len(lens) - 1, C0, sample, 1, 4, 10)
    assert e.value.code == w.EINVAL and "document id" in e.value.msg
    with pytest.raises(w.WarpError):
        w.build_index(Xt, Dt, len(lens), C0, sample, 1, 3, 10)


def test_build_names_the_first_refused_input():
    import torch

    import paper_2501_17788_amd as w

    data, X, docs, lens = _inputs(41, n_docs=200, max_len=12, n_c=200)
    sample = w.sample_passages(lens, c=20.0, seed=1)
    C0 = w.initial_centroids(X, sample, 200, seed=2)
    Xt, Dt = torch.from_numpy(X).cuda(), torch.from_numpy(docs).cuda()
    for first, second, what in ((0, np.nan, "vector 5 is zero"), (np.inf, 0, "vector 5 is not finite"),
                                (np.nan, np.nan, "vector 5 is not finite")):
        Z = C0.copy()
        Z[5, :], Z[150, 3], Z[199, :] = first, second, 0
        with pytest.raises(w.WarpError) as e:
            w.build_index(Xt, Dt, len(lens), Z, sample, 1, 4, 10)
        assert e.value.code == w.EINVAL and what in e.value.msg
    for at in (0, 70, len(sample) - 1):
        bad = sample.copy()
        bad[at:] = -1 if at == 70 else len(X)
        with pytest.raises(w.WarpError) as e:
            w.build_index(Xt, Dt, len(lens), C0, bad, 1, 4, 10)
        assert e.value.code == w.EINVAL and f"sample id {at} " in e.value.msg


def test_build_starts_after_the_null_stream():
    """The C entry point reads its inputs after the work that is on the null stream: the inputs are
    copied into place behind a few tens of milliseconds of other work, with no synchronisation
    before the call. (What the buffers hold before are other inputs, usable as well.)"""
    import ctypes

    import torch

    import paper_2501_17788_amd as w

    data, X, docs, lens = _inputs(43, n_docs=300, max_len=20, n_c=32)
    sample = w.sample_passages(lens, c=6.0, seed=1)
    C0 = w.initial_centroids(X, sample, 32, seed=2)
    want = oracle.build_index(X, docs, C0, sample, 2, 4, 500)
    assert torch.cuda.current_stream().cuda_stream == 0
    new = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (X, docs, C0, sample)]
    x, d, c0, s = (a.flip(0).contiguous() for a in new)
    n, n_c = len(X), len(C0)
    outs = [torch.empty(shape, dtype=dt, device="cuda") for shape, dt in
            (((n_c, 128), torch.float32), ((n_c + 1,), torch.int64), ((n,), torch.int32), ((n, 64), torch.uint8),
             ((16,), torch.float32), ((15,), torch.float32), ((n,), torch.int32))]
    big = torch.ones((8192, 8192), device="cuda")
    torch.cuda.synchronize()
    say("[build behind other work]")
    for _ in range(4):
        torch.mm(big, big)
    for dst, src in zip((x, d, c0, s), new):
        dst.copy_(src)
    P = ctypes.c_void_p
    rc = w.lib.warp_build_index(P(x.data_ptr()), P(d.data_ptr()), n, len(lens), P(c0.data_ptr()), n_c, P(s.data_ptr()),
                                len(sample), 2, 4, 500, *(P(o.data_ptr()) for o in outs))
    assert rc == 0, w.last_error()
    for o, key in zip(outs, ("centroids", "offsets", "doc_ids", "codes", "weights", "cutoffs", "assign")):
        np.testing.assert_array_equal(o.cpu().numpy(), want[key], err_msg=key)


def test_refused_build_leaves_the_outputs_alone():
    """Every refusal of an input comes before the first output is written, also with the starting
    vectors in the buffer of the centroids."""
    import ctypes

    import torch

    import paper_2501_17788_amd as w

    data, X, docs, lens = _inputs(41, n_docs=50, max_len=6, n_c=16)
    sample = w.sample_passages(lens, c=5.0, seed=1)
    C0 = w.initial_centroids(X, sample, 16, seed=2)
    zero, nan, out_of_range = C0.copy(), C0.copy(), sample.copy()
    zero[2], nan[3, 4], out_of_range[0] = 0, np.nan, len(X)
    n, P = len(X), ctypes.c_void_p
    for label, x, n_docs, c0, s in (("zero", X, len(lens), zero, sample), ("not finite", X, len(lens), nan, sample),
                                    ("sample id", X, len(lens), C0, out_of_range), ("norm", X * 1.5, len(lens), C0, sample),
                                    ("document id", X, len(lens) - 1, C0, sample)):
        for overlap in (False, True):
            say(f"[refused build] {label} overlap={overlap}")
            xt, dt, ct, st = (torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (x, docs, c0, s))
            cen = ct if overlap else torch.full_like(ct, 7.0)
            outs = [cen] + [torch.full(shape, 7, dtype=t, device="cuda") for shape, t in
                            (((17,), torch.int64), ((n,), torch.int32), ((n, 64), torch.uint8), ((16,), torch.float32),
                             ((15,), torch.float32), ((n,), torch.int32))]
            before = [o.clone() for o in outs]
            rc = w.lib.warp_build_index(P(xt.data_ptr()), P(dt.data_ptr()), n, n_docs, P(ct.data_ptr()), 16,
                                        P(st.data_ptr()), len(s), 1, 4, 10, *(P(o.data_ptr()) for o in outs))
            assert rc == w.EINVAL and label in w.last_error()
            for o, b in zip(outs, before):
                np.testing.assert_array_equal(o.cpu().numpy(), b.cpu().numpy(), err_msg=label)


def test_search_over_device_built_index():
    import torch

    import paper_2501_17788_amd as w

    data, X, docs, lens = _inputs(42, n_docs=800, max_len=40, n_c=128)
    sample = w.sample_passages(lens, c=12.0, seed=3)
    C0 = w.initial_centroids(X, sample, 128, seed=4)
    built = w.build_index(torch.from_numpy(X).cuda(), torch.from_numpy(docs).cuda(), len(lens), C0, sample, 4, 4,
                          3000)
    with w.Index.from_device(built["centroids"], built["offsets"], built["doc_ids"], built["codes"], 4,
                             built["weights"], len(lens)) as ix:
        got = ix.search_debug(data.queries, 16, 2000, 50)
    b = {k: v.cpu().numpy() for k, v in built.items()}
    want = oracle.search(b["centroids"], b["offsets"], b["doc_ids"], b["codes"], 4, b["weights"], len(lens),
                         data.queries, 16, 2000, 50)
    for key in ("ids", "fixed", "counts", "sel", "m_fixed", "cand_bitmap", "n_scored"):
        assert np.array_equal(got[key], want[key]), key
    hit = float(np.mean(got["ids"][:, 0] == data.query_targets))
    say(f"device-built index: target document first for {hit:.0%} of {len(data.queries)} queries")
    assert hit >= 0.5
