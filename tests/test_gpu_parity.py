"""GPU parity: the HIP path, called through the C ABI, against the fp64 dense
oracle on the same seeded inputs, element by element.

Tolerances (see tests/helpers.py): relative L2 error <= 1e-5 per output vector
for fp32 outputs; hash buckets exact outside a 1e-5 relative near-tie band.
"""
import math
import sys

import numpy as np
import pytest

from helpers import HASH_BAND, REL_L2_TOL, check_hash_against_projection, rel_l2_first_m, rel_l2_per_vector
from paper_1610_06209_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1610_06209_amd import binding

    class G:
        pass

    g = G()
    g.torch = torch
    g.b = binding
    g.dev = torch.device("cuda:0")
    return g


@pytest.fixture(autouse=True)
def _announce(request):
    print("\n[gpu-case] %s" % request.node.nodeid, file=sys.stderr, flush=True)
    yield


def _rng_case(n, batch, seed, gaussian_d3=False):
    rng = np.random.default_rng(seed)
    x = rng.standard_normal((batch, n)).astype(np.float32)
    d = (1.0 - 2.0 * rng.integers(0, 2, (3, n))).astype(np.float32)
    if gaussian_d3:
        d[2] = rng.standard_normal(n).astype(np.float32)
    return x, d


def _to(g, a):
    return g.torch.from_numpy(np.ascontiguousarray(a)).to(g.dev)


def _run_apply(g, x, d, m, epilogue, scale, **kw):
    out = g.b.spinner_apply(_to(g, x), _to(g, d[0]), _to(g, d[1]), _to(g, d[2]), m, epilogue, scale, **kw)
    g.torch.cuda.synchronize()
    return out.cpu().numpy()


# ------------------------------------------------------------------ fused sizes, plain spinner
@pytest.mark.parametrize("log2n", list(range(4, 17)))
def test_plain_spinner_every_fused_size(gpu, oracle, log2n):
    n = 1 << log2n
    # ragged batch: not a multiple of the vectors a workgroup handles, several workgroups
    batch = {4: 1000, 5: 777, 6: 333, 7: 200, 15: 5, 16: 3}.get(log2n, 37 if log2n < 12 else 9)
    x, d = _rng_case(n, batch, 1000 + log2n, gaussian_d3=(log2n % 2 == 0))
    got = _run_apply(gpu, x, d, n, "none", 1.0)
    want = oracle.apply(x, d[0], d[1], d[2], n, "none", 1.0)
    err = rel_l2_per_vector(got, want)
    assert got.shape == (batch, n)
    assert err.max() <= REL_L2_TOL, (log2n, err.max())


def test_batch_of_one_and_exact_multiple(gpu, oracle):
    for n, batch in ((256, 1), (256, 64), (1024, 16), (4096, 4), (4096, 1), (8192, 1), (8192, 2)):
        x, d = _rng_case(n, batch, n + batch)
        got = _run_apply(gpu, x, d, n, "none", 1.0)
        want = oracle.apply(x, d[0], d[1], d[2], n, "none", 1.0)
        assert rel_l2_per_vector(got, want).max() <= REL_L2_TOL


def test_empty_batch_is_a_noop(gpu):
    t = gpu.torch
    x = t.empty((0, 256), dtype=t.float32, device=gpu.dev)
    d = t.ones(256, dtype=t.float32, device=gpu.dev)
    out = gpu.b.spinner_apply(x, d, d, d)
    assert out.shape == (0, 256)
    idx = gpu.b.spinner_hash(x, t.ones((2, 3, 256), dtype=t.float32, device=gpu.dev))
    assert idx.shape == (0, 2)


def test_identity_diagonals_and_special_inputs(gpu):
    # D = I: y = H x.  x = ones -> sqrt(n) e_0 ; x = e_j -> column j of H (all +-1/sqrt(n)).
    t = gpu.torch
    for n in (64, 1024, 8192):
        one = t.ones(n, dtype=t.float32, device=gpu.dev)
        x = t.zeros((3, n), dtype=t.float32, device=gpu.dev)
        x[0] = 1.0
        x[1, 5] = 1.0
        x[2, n - 1] = 2.0
        y = gpu.b.spinner_apply(x, one, one, one).cpu().numpy().astype(np.float64)
        want0 = np.zeros(n)
        want0[0] = math.sqrt(n)
        assert np.allclose(y[0], want0, atol=1e-4 * math.sqrt(n))
        j = np.arange(n)
        col5 = np.array([(-1.0) ** bin(i & 5).count("1") for i in j]) / math.sqrt(n)
        assert np.allclose(y[1], col5, rtol=1e-6, atol=0)
        coln = 2.0 * np.array([(-1.0) ** bin(i & (n - 1)).count("1") for i in j]) / math.sqrt(n)
        assert np.allclose(y[2], coln, rtol=1e-6, atol=0)


def test_in_place_and_non_default_stream(gpu, oracle):
    t = gpu.torch
    n, batch = 2048, 11
    x, d = _rng_case(n, batch, 4242)
    want = oracle.apply(x, d[0], d[1], d[2], n, "none", 1.0)
    xd = _to(gpu, x)
    dd = [_to(gpu, d[k]) for k in range(3)]
    s = t.cuda.Stream()
    s.wait_stream(t.cuda.current_stream())
    with t.cuda.stream(s):
        gpu.b.spinner_apply(xd, dd[0], dd[1], dd[2], out=xd)        # out aliases x
    s.synchronize()
    assert rel_l2_per_vector(xd.cpu().numpy(), want).max() <= REL_L2_TOL
    # in place where a workgroup carries two vectors through the rounds (fp32 diagonals at n = 2^12, 2^13), odd batch
    for n2 in (4096, 8192):
        x, d = _rng_case(n2, 5, 4243 + n2, gaussian_d3=True)
        want = oracle.apply(x, d[0], d[1], d[2], n2, "none", 0.5)
        xd = _to(gpu, x)
        gpu.b.spinner_apply(xd, _to(gpu, d[0]), _to(gpu, d[1]), _to(gpu, d[2]), n2, "none", 0.5, out=xd)
        t.cuda.synchronize()
        assert rel_l2_per_vector(xd.cpu().numpy(), want).max() <= REL_L2_TOL


# ------------------------------------------------------------------ truncation
@pytest.mark.parametrize("n,m,scale", [(256, 64, 2.0), (256, 5, 1.0), (1024, 1000, 0.5), (4096, 1, 1.0),
                                       (16384, 1024, 4.0), (8192, 4100, 1.0), (64, 62, 3.0)])
def test_first_m_rows(gpu, oracle, n, m, scale):
    x, d = _rng_case(n, 7, n + m)
    got = _run_apply(gpu, x, d, m, "none", scale)
    want = oracle.apply(x, d[0], d[1], d[2], m, "none", scale)
    assert got.shape == (7, m)
    assert rel_l2_first_m(got, want, x, n, m, scale).max() <= REL_L2_TOL


@pytest.mark.parametrize("log2n", list(range(8, 17)))
def test_first_m_rows_with_pruned_last_round(gpu, oracle, log2n):
    # m <= n/16 takes the kernels whose last round only forms the sums it needs on the four
    # highest index bits; both diagonal forms, exact and ragged m.
    n = 1 << log2n
    batch = 21 if log2n < 12 else 5
    w = W.Workload("p", "apply", n, batch, n, "none", 1.0, 1, "normal_heavy", 8800 + log2n, batch)
    x = W.make_x_numpy(w)
    ds = W.diag_sets(w)
    xd, dsd = _to(gpu, x), _to(gpu, ds)
    signs = gpu.b.spinner_pack_signs(dsd)
    y = oracle.spinner(x, ds[0, 0], ds[0, 1], ds[0, 2])

    def check(got, want, m, scale, what):
        assert got.shape == (batch, m)
        err = rel_l2_first_m(got, want, x, n, m, scale)
        assert err.max() <= REL_L2_TOL, (log2n, m, what, err.max())

    for m in (n // 16, n // 16 - 3, n // 64, 1, n // 16 + 1):
        scale = math.sqrt(n / m)
        want = oracle.epilogue_none(y, m, scale)
        check(gpu.b.spinner_apply(xd, dsd[0, 0], dsd[0, 1], dsd[0, 2], m, "none", scale).cpu().numpy(), want, m, scale,
              "fp32 diagonals")
        check(gpu.b.spinner_apply_signs(xd, signs, m, "none", scale).cpu().numpy(), want, m, scale, "sign words")


@pytest.mark.parametrize("log2n,pruned", [(13, True), (14, True), (16, True), (16, False)])
def test_first_m_rows_with_diagonals_in_flight_ahead(gpu, oracle, log2n, pruned):
    # every entry of every diagonal another value: one that meets the wrong coordinate, or meets it twice, shows
    n = 1 << log2n
    rng = np.random.default_rng(1900 + log2n + pruned)
    d = (rng.standard_normal((3, n)) * 0.5 + 1.0).astype(np.float32)
    for m, batch in ((n // 16, 3), (n // 16 - 3, 2), (n // 64, 2)) if pruned else ((n - 1, 2), (n // 2, 3), (n, 49)):
        x = rng.standard_normal((batch, n)).astype(np.float32)
        got = _run_apply(gpu, x, d, m, "none", 1.0)
        if batch > 3:                                   # the kernel for more than a few vectors, checked on the last
            x, got = x[-2:], got[-2:]
        want = oracle.apply(x, d[0], d[1], d[2], m, "none", 1.0)
        assert rel_l2_per_vector(got, want).max() <= REL_L2_TOL, (m, batch)


# ------------------------------------------------------------------ random features
@pytest.mark.parametrize("n,m,scale", [(64, 64, 8.0), (1024, 1024, 32.0), (1024, 100, 3.0), (4096, 4096, 64.0),
                                       (16384, 16384, 1.0)])
def test_cos_sin_features(gpu, oracle, n, m, scale):
    x, d = _rng_case(n, 6, 7 * n + m)
    got = _run_apply(gpu, x, d, m, "cossin", scale)
    want = oracle.apply(x, d[0], d[1], d[2], m, "cossin", scale)
    assert got.shape == (6, 2 * m)
    err = rel_l2_per_vector(got, want)
    assert err.max() <= REL_L2_TOL, err.max()
    assert np.allclose(np.linalg.norm(got.astype(np.float64), axis=1), 1.0, atol=1e-5)


# ------------------------------------------------------------------ hash
@pytest.mark.parametrize("log2n", list(range(4, 17)))
def test_hash_every_size(gpu, oracle, log2n):
    n = 1 << log2n
    batch = 70 if log2n < 12 else 6
    L = 3
    w = W.Workload("h", "hash", n, batch, n, "hash", 1.0, L, "unit_normal", 500 + log2n, batch)
    x = W.make_x_numpy(w)
    ds = W.diag_sets(w)
    got = gpu.b.spinner_hash(_to(gpu, x), _to(gpu, ds)).cpu().numpy()
    assert got.shape == (batch, L) and got.dtype == np.int32
    _, ys = oracle.hash(x, ds, return_y=True)
    exact, banded = check_hash_against_projection(got, ys)
    assert exact + banded == batch * L
    assert banded <= 1
    if log2n > 14:      # one launch per triple: also from packed sign words (the smaller sizes: test_sign_word_path_every_fused_size)
        signs = gpu.b.spinner_pack_signs(_to(gpu, ds))
        got = gpu.b.spinner_hash_signs(_to(gpu, x), signs, L).cpu().numpy()
        exact, banded = check_hash_against_projection(got, ys)
        assert exact + banded == batch * L and banded <= 1


@pytest.mark.parametrize("log2n,batch,L", [(17, 5, 2), (18, 3, 1), (20, 2, 2), (22, 1, 1)])
def test_hash_above_the_fused_range(gpu, oracle, log2n, batch, L):
    # four passes per triple into the workspace, then the bucket from there (spinner_hash_ws); both diagonal forms
    n = 1 << log2n
    w = W.Workload("h", "hash", n, batch, n, "hash", 1.0, L, "unit_normal", 600 + log2n, batch)
    x = W.make_x_numpy(w)
    ds = W.diag_sets(w)
    ys = np.stack([oracle.spinner_by_products(x, ds[l, 0], ds[l, 1], ds[l, 2]) for l in range(L)])
    got = gpu.b.spinner_hash_ws(_to(gpu, x), _to(gpu, ds)).cpu().numpy()
    assert got.shape == (batch, L) and got.dtype == np.int32
    exact, banded = check_hash_against_projection(got, ys)
    assert exact + banded == batch * L and banded <= 1
    signs = gpu.b.spinner_pack_signs(_to(gpu, ds))
    got = gpu.b.spinner_hash_signs_ws(_to(gpu, x), signs, L).cpu().numpy()
    exact, banded = check_hash_against_projection(got, ys)
    assert exact + banded == batch * L and banded <= 1
    with pytest.raises(gpu.b.SpinnerError):
        gpu.b.spinner_hash(_to(gpu, x), _to(gpu, ds))      # the call without a workspace stops at 2^16


def test_hash_with_workspace_is_the_plain_call_up_to_the_fused_range(gpu):
    # up to 2^16 the variant with a workspace argument is spinner_hash itself: no workspace needed, same buckets
    t = gpu.torch
    for n, batch in ((1024, 300), (1 << 15, 5)):
        w = W.Workload("h", "hash", n, batch, n, "hash", 1.0, 3, "unit_normal", 640 + n, batch)
        x, ds = _to(gpu, W.make_x_numpy(w)), _to(gpu, W.diag_sets(w))
        assert gpu.b.spinner_hash_workspace_bytes(n, batch) == 0
        assert t.equal(gpu.b.spinner_hash_ws(x, ds), gpu.b.spinner_hash(x, ds))
        signs = gpu.b.spinner_pack_signs(ds)
        assert t.equal(gpu.b.spinner_hash_signs_ws(x, signs, 3), gpu.b.spinner_hash_signs(x, signs, 3))


def test_hash_above_the_fused_range_in_several_slices(gpu):
    # n = 2^17, 513 vectors: the passes walk the batch in two slices (257 + 256).  The bucket must be the argmax of the
    # projection that spinner_apply writes for the same triple (same passes, so the same bits; random data has no ties)
    t = gpu.torch
    n, batch, L = 1 << 17, 513, 2
    g = t.Generator(device=gpu.dev)
    g.manual_seed(77)
    x = t.randn((batch, n), generator=g, device=gpu.dev, dtype=t.float32)
    ds = (1.0 - 2.0 * t.randint(0, 2, (L, 3, n), generator=g, device=gpu.dev)).float()
    idx = gpu.b.spinner_hash_ws(x, ds)
    for l in range(L):
        y = gpu.b.spinner_apply(x, ds[l, 0], ds[l, 1], ds[l, 2])
        i = y.abs().argmax(dim=1)
        want = i + n * (y[t.arange(batch, device=gpu.dev), i] < 0).long()
        assert bool((idx[:, l].long() == want).all()), l


def test_hash_above_the_fused_range_on_constructed_inputs(gpu):
    # D = I: x = +-(column j of normalised H) gives y = +-e_j exactly (entries are +-2^-9 at n = 2^18); a tie between
    # two coordinates that fall into different chunks of the scan goes to the lower index; zero vector -> bucket 0
    t = gpu.torch
    n = 1 << 18
    ones = t.ones((1, 3, n), dtype=t.float32, device=gpu.dev)
    i = np.arange(n, dtype=np.int64)

    def col(j):
        v, par = i & j, np.zeros(n, dtype=np.int64)
        for s in range(18):
            par ^= (v >> s) & 1
        return ((1.0 - 2.0 * par) / 512.0).astype(np.float32)

    js = [0, 3, 65535, 65536, 200000, n - 1]
    x = np.zeros((2 * len(js) + 3, n), dtype=np.float32)
    for k, j in enumerate(js):
        x[2 * k] = col(j)
        x[2 * k + 1] = -col(j)
    x[-3] = col(70000) + col(5)            # tie across chunks: lowest index
    x[-2] = -col(262000) - col(131072)     # tie of two negative coordinates
    got = gpu.b.spinner_hash_ws(_to(gpu, x), ones).cpu().numpy()[:, 0]
    for k, j in enumerate(js):
        assert got[2 * k] == j and got[2 * k + 1] == j + n, j
    assert got[-3] == 5 and got[-2] == 131072 + n and got[-1] == 0


@pytest.mark.parametrize("n", [256, 1024])
def test_hash_from_sign_words_on_constructed_inputs(gpu, n):
    # D = I as packed words: x = H z for sums z of few unit vectors gives y = z exactly (entries are multiples of a power of
    # two).  Several vectors share a wave and are searched together: maxima in every group of registers, at the ends, of
    # either sign, exact ties across registers, lanes and signs (lowest index), the zero vector, a NaN vector (bucket 0)
    t = gpu.torch
    i = np.arange(n)
    H = 1.0 - 2.0 * (np.array([bin(v).count("1") & 1 for v in range(n)])[i[:, None] & i[None]])
    z, want = [], []
    for j in list(range(0, n, 37)) + [n - 1]:
        for s in (1.0, -1.0):
            row = np.zeros(n); row[j] = s; z.append(row); want.append(j + (n if s < 0 else 0))
    rng = np.random.default_rng(n)
    for _ in range(60):
        at = np.sort(rng.choice(n, 4, replace=False))
        val = rng.choice([-1.0, 1.0], 4)
        row = np.zeros(n); row[at] = val; z.append(row); want.append(at[0] + (n if val[0] < 0 else 0))
    z.append(np.zeros(n)); want.append(0)
    x = (np.array(z) @ H / math.sqrt(n)).astype(np.float32)
    x = np.concatenate([x, np.full((1, n), np.nan, dtype=np.float32), x[:3]])
    want = np.array(want + [0] + want[:3])
    assert len(want) % 4                                       # the last wave is not full
    signs = gpu.b.spinner_pack_signs(t.ones((2, 3, n), dtype=t.float32, device=gpu.dev))
    got = gpu.b.spinner_hash_signs(_to(gpu, x), signs, 2).cpu().numpy()
    assert np.array_equal(got, np.stack([want, want], 1))


@pytest.mark.parametrize("n", [256, 1024])
def test_hash_of_vectors_that_overflow_is_the_same_from_sign_words(gpu, n):
    # D = I and x = (z / n) with z = 2^127 at 0, 1, n/2, n/2 + 1 and -2^127 two places further on: two transforms give z exactly, and
    # the third adds +inf and -inf into coordinate 0 whatever the order of its stages, so y_0 is NaN, half of the rest +-inf or NaN
    # and half 0.  A NaN in the first coordinate is kept (numpy's argmax does the same): bucket 0 from either form of the
    # diagonals, and the vector beside it in the same wave keeps its own
    t = gpu.torch
    z = np.zeros(n)
    z[[0, 1, n // 2, n // 2 + 1]] = 2.0 ** 127
    z[[2, 3, n // 2 + 2, n // 2 + 3]] = -(2.0 ** 127)
    rng = np.random.default_rng(n)
    x = rng.standard_normal((7, n)).astype(np.float32)
    x[[0, 3, 6]] = (z / n).astype(np.float32)
    ones = t.ones((1, 3, n), dtype=t.float32, device=gpu.dev)
    x = _to(gpu, x)
    from_fp32 = gpu.b.spinner_hash(x, ones).cpu().numpy()[:, 0]
    from_words = gpu.b.spinner_hash_signs(x, gpu.b.spinner_pack_signs(ones), 1).cpu().numpy()[:, 0]
    assert list(from_fp32[[0, 3, 6]]) == [0, 0, 0]
    assert np.array_equal(from_words, from_fp32)


def test_hash_rules_on_constructed_inputs(gpu):
    # D = I, x = +-(column j of normalised H)  ->  bucket j / j + n ; zero vector -> bucket 0 ;
    # exact tie -> lowest index.
    t = gpu.torch
    n = 1024
    ones = t.ones((2, 3, n), dtype=t.float32, device=gpu.dev)
    js = [0, 1, 77, 512, n - 1]
    x = np.zeros((2 * len(js) + 2, n), dtype=np.float32)
    for k, j in enumerate(js):
        col = np.array([(-1.0) ** bin(i & j).count("1") for i in range(n)]) / 32.0     # sqrt(1024) = 32, exact
        x[2 * k] = col
        x[2 * k + 1] = -col
    # x = e_0 + e_3 gives y = H x with |y_i| = 2/sqrt(n) on a quarter of the coordinates... use a
    # cleaner tie: x = H(e_5 + e_9) so that y = e_5 + e_9 exactly (entries are multiples of 1/32)
    c5 = np.array([(-1.0) ** bin(i & 5).count("1") for i in range(n)]) / 32.0
    c9 = np.array([(-1.0) ** bin(i & 9).count("1") for i in range(n)]) / 32.0
    x[-2] = c5 + c9
    got = gpu.b.spinner_hash(_to(gpu, x), ones).cpu().numpy()
    for k, j in enumerate(js):
        assert got[2 * k].tolist() == [j, j]
        assert got[2 * k + 1].tolist() == [j + n, j + n]
    assert got[-2].tolist() == [5, 5]            # tie between 5 and 9 -> lowest index
    assert got[-1].tolist() == [0, 0]            # all-zero vector


def test_hash_antipodal_symmetry_full_gpu(gpu):
    w = W.Workload("h", "hash", 512, 4096, 512, "hash", 1.0, 5, "unit_normal", 31, 0)
    x = _to(gpu, W.make_x_numpy(w))
    ds = _to(gpu, W.diag_sets(w))
    h = gpu.b.spinner_hash(x, ds)
    hn = gpu.b.spinner_hash(-x, ds)
    assert bool(((h + w.n) % (2 * w.n) == hn).all())
    assert int(h.min()) >= 0 and int(h.max()) < 2 * w.n


# ------------------------------------------------------------------ n above the fused range (four passes)
@pytest.mark.parametrize("log2n,batch", [(15, 3), (16, 2), (18, 2), (20, 2), (21, 1)])
def test_multipass_plain(gpu, oracle, log2n, batch):
    n = 1 << log2n
    x, d = _rng_case(n, batch, 900 + log2n, gaussian_d3=(log2n == 16))
    got = _run_apply(gpu, x, d, n, "none", 1.0)
    want = oracle.apply(x, d[0], d[1], d[2], n, "none", 1.0)
    assert rel_l2_per_vector(got, want).max() <= REL_L2_TOL


@pytest.mark.parametrize("log2n,batch", [(22, 2), (23, 1), (24, 1)])
def test_multipass_largest_sizes_against_the_oracle(gpu, oracle, log2n, batch):
    # The plain-loop oracle takes minutes per vector here; its route through two dense matrix products per round
    # (pinned on the CPU against the plain loops) takes seconds.  Random +-1 first and second diagonals, Gaussian
    # third diagonal through spinner_apply; +-1 diagonals through both forms, full width and the first rows.
    n = 1 << log2n
    x, d = _rng_case(n, batch, 2200 + log2n, gaussian_d3=True)
    got = _run_apply(gpu, x, d, n, "none", 1.0)
    want = oracle.spinner_by_products(x, d[0], d[1], d[2])
    assert rel_l2_per_vector(got, want).max() <= REL_L2_TOL
    del got
    x, d = _rng_case(n, batch, 2300 + log2n)
    want = oracle.spinner_by_products(x, d[0], d[1], d[2])
    xd = _to(gpu, x)
    signs = gpu.b.spinner_pack_signs(_to(gpu, d[None, :, :]))
    got = gpu.b.spinner_apply_signs(xd, signs).cpu().numpy()
    assert rel_l2_per_vector(got, want).max() <= REL_L2_TOL
    m = 3000
    got = gpu.b.spinner_apply_signs(xd, signs, m, "none", 2.0).cpu().numpy()
    assert rel_l2_first_m(got, 2.0 * want[:, :m], x, n, m, 2.0).max() <= REL_L2_TOL
    got = _run_apply(gpu, x, d, m, "none", 2.0)
    assert rel_l2_first_m(got, 2.0 * want[:, :m], x, n, m, 2.0).max() <= REL_L2_TOL


@pytest.mark.parametrize("log2n", [19, 22, 23, 24])
def test_multipass_largest_sizes_by_properties(gpu, log2n):
    # The O(n^2)-per-factor oracle takes minutes per vector here, so these sizes are checked by
    # what holds at any size: (a) D = I maps e_j to column j of H, entry (-1)^popcount(i&j)/sqrt(n);
    # (b) for +-1 diagonals the product is orthogonal and H D2 H D3 H (H D3 H D2 H D1 x) = D1 x,
    # so a second call with diagonals (1, d3, d2) must return D1 x; (c) the norm is preserved.
    # n = 2^19 is also covered by the oracle-backed sizes around it and ties the two kinds of check.
    t = gpu.torch
    n = 1 << log2n
    one = t.ones(n, dtype=t.float32, device=gpu.dev)
    js = [0, 1, 12345 % n, n // 2 + 77, n - 1]
    x = t.zeros((len(js), n), dtype=t.float32, device=gpu.dev)
    for k, j in enumerate(js):
        x[k, j] = 1.0
    y = gpu.b.spinner_apply(x, one, one, one)
    idx = t.arange(n, device=gpu.dev, dtype=t.int64)
    for k, j in enumerate(js):
        v = idx & j
        par = t.zeros_like(v)
        for sft in range(log2n):
            par ^= (v >> sft) & 1
        want = (1.0 - 2.0 * par.double()) / math.sqrt(n)
        assert float((y[k].double() - want).abs().max()) <= 1e-6 / math.sqrt(n) * 4 + 1e-12, (log2n, j)
    del x, y
    g = t.Generator(device=gpu.dev)
    g.manual_seed(99 + log2n)
    xr = t.randn((2, n), generator=g, device=gpu.dev, dtype=t.float32)
    d = (1.0 - 2.0 * t.randint(0, 2, (3, n), generator=g, device=gpu.dev)).float()
    yr = gpu.b.spinner_apply(xr, d[0], d[1], d[2])
    nx, ny = xr.double().norm(dim=1), yr.double().norm(dim=1)
    assert float(((ny / nx) - 1).abs().max()) < 1e-5
    z = gpu.b.spinner_apply(yr, one, d[2], d[1])
    err = ((z * d[0]).double() - xr.double()).norm(dim=1) / nx
    assert float(err.max()) < 1e-5, float(err.max())
    # the same through packed sign words (row passes by the words of their tile, column pass by its lane masks, each
    # with the tile geometry of this size): equal to the fp32-diagonal result up to rounding, and inverted the same way
    signs = gpu.b.spinner_pack_signs(d[None].contiguous())
    ys = gpu.b.spinner_apply_signs(xr, signs)
    assert float(((ys.double() - yr.double()).norm(dim=1) / ny).max()) < 1e-6
    back = gpu.b.spinner_pack_signs(t.stack([one, d[2], d[1]])[None].contiguous())
    zs = gpu.b.spinner_apply_signs(ys, back)
    err = ((zs * d[0]).double() - xr.double()).norm(dim=1) / nx
    assert float(err.max()) < 1e-5, float(err.max())


def test_multipass_truncated_and_features(gpu, oracle):
    n = 1 << 15
    x, d = _rng_case(n, 3, 77)
    y = oracle.spinner(x, d[0], d[1], d[2])
    got = _run_apply(gpu, x, d, 1024, "none", 4.0)
    assert got.shape == (3, 1024)
    assert rel_l2_per_vector(got, oracle.epilogue_none(y, 1024, 4.0)).max() <= REL_L2_TOL
    got = _run_apply(gpu, x, d, 2048, "cossin", 2.0)
    assert got.shape == (3, 4096)
    assert rel_l2_per_vector(got, oracle.epilogue_cossin(y, 2048, 2.0)).max() <= REL_L2_TOL


def test_multipass_ragged_last_slice(gpu, oracle):
    # The four-pass schedule walks the batch in equal slices of at most 256 MiB; a batch that does not divide leaves a
    # shorter last slice (n = 2^17: 513 vectors are 257 + 256).  First and last row of each slice against the oracle,
    # for an output narrower than n (passes run in the workspace) and for features, with both diagonal forms.
    t = gpu.torch
    n, batch = 1 << 17, 513
    rows = [0, 256, 257, 512]
    g = t.Generator(device=gpu.dev)
    g.manual_seed(4171)
    xd = t.randn((batch, n), generator=g, device=gpu.dev, dtype=t.float32)
    d = W.rademacher_diagonals(n, 3, 4172)
    dd = [_to(gpu, d[k]) for k in range(3)]
    x = xd[rows].cpu().numpy()                                   # the bits the GPU consumed
    y = oracle.spinner(x, d[0], d[1], d[2])
    signs = gpu.b.spinner_pack_signs(_to(gpu, d[None]))
    m = 1000
    for form in ("fp32", "signs"):
        if form == "fp32":
            got = gpu.b.spinner_apply(xd, dd[0], dd[1], dd[2], m, "none", 3.0)
        else:
            got = gpu.b.spinner_apply_signs(xd, signs, m, "none", 3.0)
        assert got.shape == (batch, m)
        assert rel_l2_per_vector(got[rows].cpu().numpy(), oracle.epilogue_none(y, m, 3.0)).max() <= REL_L2_TOL, form
        del got
        if form == "fp32":
            got = gpu.b.spinner_apply(xd, dd[0], dd[1], dd[2], 512, "cossin", 0.05)
        else:
            got = gpu.b.spinner_apply_signs(xd, signs, 512, "cossin", 0.05)
        assert got.shape == (batch, 1024)
        assert rel_l2_per_vector(got[rows].cpu().numpy(), oracle.epilogue_cossin(y, 512, 0.05)).max() <= REL_L2_TOL, form
        del got


def test_features_above_the_fused_range_at_the_kernel_scale(gpu, oracle):
    # Above n = 2^14 the feature map runs on fp32 butterflies (four passes; the fused sizes compute in fp64).  With
    # scale = sqrt(n) / sigma (Section 5) the angles w are as large as |x|, and 3 log2 n fp32 roundings leave an
    # error of about 3.4e-8 * sqrt(3 log2 n) * rms(w) radians in each of them, which is also the relative error of
    # the unit-norm feature vector: beyond 1e-5 once rms(w) exceeds about 40.  The header states this bound
    # (relative error <= 5e-7 * rms(w), at least 1e-5); this case pins it at n = 2^15.
    n, batch = 1 << 15, 4
    x, d = _rng_case(n, batch, 1515)                             # N(0,1) entries: |x| = 181
    scale = math.sqrt(n)
    y = oracle.spinner(x, d[0], d[1], d[2])
    want = oracle.epilogue_cossin(y, n, scale)
    rms_w = scale * np.linalg.norm(y, axis=1) / math.sqrt(n)
    bound = np.maximum(1e-5, 5e-7 * rms_w)
    got = _run_apply(gpu, x, d, n, "cossin", scale)
    err = rel_l2_per_vector(got, want)
    assert (err <= bound).all(), (err, bound)
    signs = gpu.b.spinner_pack_signs(_to(gpu, d[None]))
    got = gpu.b.spinner_apply_signs(_to(gpu, x), signs, n, "cossin", scale).cpu().numpy()
    err = rel_l2_per_vector(got, want)
    assert (err <= bound).all(), (err, bound)
    # small angles (rms(w) = 8): inside the plain tolerance
    got = _run_apply(gpu, x, d, n, "cossin", scale / 22.6)
    assert rel_l2_per_vector(got, oracle.epilogue_cossin(y, n, scale / 22.6)).max() <= REL_L2_TOL


@pytest.mark.parametrize("log2n,few", [(15, 32), (16, 48)])
def test_few_and_many_vectors_of_the_widest_fused_sizes(gpu, oracle, log2n, few):
    # n = 2^15, 2^16: up to 32 vectors (features at 2^16: 48) go through the four passes, more through one fused kernel.  The
    # same vectors on both sides of the limit, some against the oracle, in place, on both diagonal forms, and features of rows
    # of whole 16-byte pieces and others, alone and in stacked blocks
    t, n = gpu.torch, 1 << log2n
    x, d = _rng_case(n, 2, 1600 + log2n)
    g = t.Generator(device=gpu.dev)
    g.manual_seed(log2n)
    xd = t.randn((few + 1, n), generator=g, device=gpu.dev)
    xd[:2] = _to(gpu, x)
    dd = [_to(gpu, d[k]) for k in range(3)]
    signs = gpu.b.spinner_pack_signs(_to(gpu, d[None]))
    y = oracle.spinner(x, d[0], d[1], d[2])
    for f in (lambda v, m, e, c: gpu.b.spinner_apply(v, *dd, m, e, c), lambda v, m, e, c: gpu.b.spinner_apply_signs(v, signs, m, e, c)):
        for k in (1, 32, 33):
            got = f(xd[:k], n, "none", 1.5)
            assert rel_l2_per_vector(got[:1].cpu().numpy(), oracle.epilogue_none(y[:1], n, 1.5)).max() <= 1e-6
            # two roundings of each of 3 log2(n) stages, in another order
            assert float((got - f(xd, n, "none", 1.5)[:k]).norm() / got.norm()) <= 1e-6
        for m in (n, 4096, 1001):
            many, less = f(xd, m, "cossin", 8.0), f(xd[:few], m, "cossin", 8.0)
            assert rel_l2_per_vector(many[:2].cpu().numpy(), oracle.epilogue_cossin(y, m, 8.0)).max() <= REL_L2_TOL
            # angles of rms 8 carry 3.4e-8 sqrt(3 log2 n) of it on either side
            assert float((many[:few] - less).norm() / less.norm()) <= 2 * 3.4e-8 * math.sqrt(3 * log2n) * 8.0
    here = xd[:5].clone()
    gpu.b.spinner_apply(here, *dd, n, "none", 1.5, out=here)
    assert t.equal(here, gpu.b.spinner_apply(xd[:5], *dd, n, "none", 1.5))
    sets = t.stack([t.stack(dd), t.stack((dd[2], dd[0], dd[1]))])
    both = gpu.b.spinner_apply_blocks(xd, sets, 512, "cossin", 8.0).reshape(few + 1, 2, 2, 512)
    for l in range(2):
        one = gpu.b.spinner_apply(xd, *sets[l], 512, "cossin", 8.0).reshape(few + 1, 2, 512) / math.sqrt(2.0)
        assert float((both[:, :, l] - one).abs().max()) <= 2.0 ** -22 / math.sqrt(2 * 512)


@pytest.mark.parametrize("log2n,few", [(15, 32), (16, 48)])
@pytest.mark.parametrize("scale", [8.0, 5.7])
def test_features_of_the_widest_fused_sizes_are_no_further_off_than_those_of_the_passes(gpu, log2n, few, scale):
    # the same vectors through the four passes, few at a time, and through the fused kernel, both against fp64: over these 2^24
    # values and more two forms with the same error differ by less than 0.1 %.  A scale that is a power of two leaves the passes' angle
    # of 2^16 without a rounding of its own
    t, n = gpu.torch, 1 << log2n
    g = t.Generator(device=gpu.dev)
    g.manual_seed(log2n)
    x = t.randn((5 * few, n), generator=g, device=gpu.dev)
    d = t.randint(0, 2, (3, n), generator=g, device=gpu.dev).float() * 2 - 1
    w = x.double()
    for k in range(3):
        w = w * d[k].double()
        for b in range(log2n):
            y = w.reshape(-1, n >> (b + 1), 2, 1 << b)
            w = t.stack((y[:, :, 0] + y[:, :, 1], y[:, :, 0] - y[:, :, 1]), 2).reshape(-1, n)
    w *= scale / n ** 1.5
    want = t.cat((t.cos(w), t.sin(w)), 1) / math.sqrt(n)
    signs = gpu.b.spinner_pack_signs(d[None].contiguous())
    for f in (lambda v: gpu.b.spinner_apply(v, *d, n, "cossin", scale), lambda v: gpu.b.spinner_apply_signs(v, signs, n, "cossin", scale)):
        passes = t.cat([f(x[i:i + few]) for i in range(0, 5 * few, few)])
        fused = f(x)
        assert float((fused - want).norm()) <= 1.001 * float((passes - want).norm())


# ------------------------------------------------------------------ +-1 diagonals as packed sign words
@pytest.mark.parametrize("log2n", list(range(4, 15)))
def test_sign_word_path_every_fused_size(gpu, oracle, log2n):
    n = 1 << log2n
    batch = {4: 1000, 5: 777, 6: 333, 7: 200}.get(log2n, 37 if log2n < 12 else 9)
    L = 2
    w = W.Workload("s", "hash", n, batch, n, "hash", 1.0, L, "normal", 7000 + log2n, batch)
    x = W.make_x_numpy(w)
    ds = W.diag_sets(w)
    xd, dsd = _to(gpu, x), _to(gpu, ds)
    signs = gpu.b.spinner_pack_signs(dsd)
    assert signs.numel() == gpu.b.spinner_signs_bytes(n, L)
    for t in range(L):                                          # plain spinner, each triple
        got = gpu.b.spinner_apply_signs(xd, signs, triple=t).cpu().numpy()
        want = oracle.apply(x, ds[t, 0], ds[t, 1], ds[t, 2], n, "none", 1.0)
        assert rel_l2_per_vector(got, want).max() <= REL_L2_TOL, (log2n, t)
    m = max(1, n // 4)
    got = gpu.b.spinner_apply_signs(xd, signs, m, "cossin", 0.75 * math.sqrt(n), triple=1).cpu().numpy()
    want = oracle.apply(x, ds[1, 0], ds[1, 1], ds[1, 2], m, "cossin", 0.75 * math.sqrt(n))
    assert rel_l2_per_vector(got, want).max() <= REL_L2_TOL
    h = gpu.b.spinner_hash_signs(xd, signs, L).cpu().numpy()
    _, ys = oracle.hash(x, ds, return_y=True)
    exact, banded = check_hash_against_projection(h, ys)
    assert exact + banded == batch * L and banded <= 1
    # the sign-word path and the fp32-diagonal path agree on +-1 diagonals: bit for bit where both use the
    # same order of butterflies (n < 2^12), to rounding above that (the sign-word kernels order them differently)
    ref = gpu.b.spinner_apply(xd, dsd[0, 0], dsd[0, 1], dsd[0, 2])
    alt = gpu.b.spinner_apply_signs(xd, signs, triple=0)
    if log2n < 12:
        assert bool((ref == alt).all())
    else:
        assert rel_l2_per_vector(alt.cpu().numpy(), ref.cpu().numpy().astype(np.float64)).max() <= 2e-6
    assert bool((gpu.b.spinner_hash(xd, dsd) == gpu.b.spinner_hash_signs(xd, signs, L)).all())


@pytest.mark.parametrize("m,scale,batch", [(4096, 64.0, 7), (1000, 48.0, 5), (64, 64.0, 2), (1, 64.0, 3)])
def test_features_from_sign_words_n4096(gpu, oracle, m, scale, batch):
    # n = 4096 with sign words runs the feature kernel that keeps every butterfly between registers:
    # odd batches (a workgroup's last wave has no vector), row limits inside and at the edge of a 64-lane run
    n = 4096
    x, d = _rng_case(n, batch, 31 * m + batch)
    ds = np.stack([d, W.rademacher_diagonals(n, 3, 77 + m)])
    signs = gpu.b.spinner_pack_signs(_to(gpu, ds))
    for t in range(2):
        got = gpu.b.spinner_apply_signs(_to(gpu, x), signs, m, "cossin", scale, triple=t).cpu().numpy()
        want = oracle.apply(x, ds[t, 0], ds[t, 1], ds[t, 2], m, "cossin", scale)
        assert got.shape == (batch, 2 * m)
        assert rel_l2_per_vector(got, want).max() <= REL_L2_TOL, (m, t)
        # the same kernel takes fp32 diagonals (multiplied, not flipped)
        got = _run_apply(gpu, x, ds[t], m, "cossin", scale)
        assert rel_l2_per_vector(got, want).max() <= REL_L2_TOL, (m, t, "fp32 diagonals")
    # diagonals that are not +-1: Gaussian third diagonal (the H D_g H D2 H D1 member), scaled first and second
    rng = np.random.default_rng(5 * m + batch)
    dg = np.stack([d[0] * np.float32(0.75), d[1] * np.float32(-1.5), rng.standard_normal(n).astype(np.float32)])
    got = _run_apply(gpu, x, dg, m, "cossin", scale / 2)
    want = oracle.apply(x, dg[0], dg[1], dg[2], m, "cossin", scale / 2)
    assert rel_l2_per_vector(got, want).max() <= REL_L2_TOL, (m, "general diagonals")


@pytest.mark.parametrize("m", [1, 33, 511, 512, 513, 992, 1001])
def test_features_n1024_rows_of_whole_lines_and_others(gpu, oracle, m):
    # n = 1024: rows of whole 128-byte lines (m a multiple of 32) and short ones (m < 512) are stored past the caches, others
    # are not; an odd batch leaves half of the last wave without a vector
    n, batch, scale = 1024, 7, 32.0
    x, d = _rng_case(n, batch, 53 * m)
    want = oracle.apply(x, d[0], d[1], d[2], m, "cossin", scale)
    got = gpu.b.spinner_apply_signs(_to(gpu, x), gpu.b.spinner_pack_signs(_to(gpu, d[None])), m, "cossin", scale).cpu().numpy()
    assert rel_l2_per_vector(got, want).max() <= REL_L2_TOL
    assert rel_l2_per_vector(_run_apply(gpu, x, d, m, "cossin", scale), want).max() <= REL_L2_TOL
    if m in (512, 992):                               # blocks: m a multiple of 4
        for mb in (m, m + 4):
            ds = np.stack([d, W.rademacher_diagonals(n, 3, 54 * m)])
            got = gpu.b.spinner_apply_blocks(_to(gpu, x), _to(gpu, ds), mb, "cossin", scale).cpu().numpy()
            assert rel_l2_per_vector(got, oracle.apply_blocks(x, ds, mb, "cossin", scale)).max() <= REL_L2_TOL


@pytest.mark.parametrize("log2n", [15, 16, 17, 18, 19, 20, 21, 22])
def test_sign_word_path_above_the_feature_and_hash_range(gpu, oracle, log2n):
    # Above 2^14 the packed form is sign words followed by the fp32 diagonals.  n = 2^15, 2^16: the words serve the fused
    # plain kernel; in the four-pass schedule (features from 2^15, everything from 2^17) the row passes flip by the
    # words of their own tile once a row fills a wave (rows of 2^9 .. 2^14 elements here, each with its own kernel
    # geometry) and the column pass flips by the lane masks that spinner_pack_signs prepared for its tiles.  Two triples, so that the per-triple stride is
    # used; three vectors, so that the tiles of one row index are an odd count.
    n = 1 << log2n
    w = W.Workload("s", "apply", n, 3, n, "none", 1.0, 2, "normal", 8100 + log2n, 3)
    x = W.make_x_numpy(w)
    ds = W.diag_sets(w)
    xd = _to(gpu, x)
    signs = gpu.b.spinner_pack_signs(_to(gpu, ds))
    assert signs.numel() == gpu.b.spinner_signs_bytes(n, 2) == 2 * gpu.b.spinner_signs_bytes(n, 1)
    # from 2^20 on the oracle's route through dense matrix products (seconds where the plain loops take a minute)
    project = oracle.spinner_by_products if log2n >= 20 else oracle.spinner
    ys = [project(x, ds[t, 0], ds[t, 1], ds[t, 2]) for t in range(2)]
    for t in range(2):
        got = gpu.b.spinner_apply_signs(xd, signs, triple=t).cpu().numpy()
        assert rel_l2_per_vector(got, oracle.epilogue_none(ys[t], n, 1.0)).max() <= REL_L2_TOL, t
    m = 512
    got = gpu.b.spinner_apply_signs(xd, signs, m, "cossin", 2.0, triple=1).cpu().numpy()
    assert rel_l2_per_vector(got, oracle.epilogue_cossin(ys[1], m, 2.0)).max() <= REL_L2_TOL
    got = gpu.b.spinner_apply_signs(xd, signs, m, "none", 3.0, triple=1).cpu().numpy()      # pruned last round
    assert rel_l2_per_vector(got, oracle.epilogue_none(ys[1], m, 3.0)).max() <= REL_L2_TOL


def test_stream_copy(gpu):
    t = gpu.torch
    src = t.randn(1 << 20, device=gpu.dev)
    dst = t.zeros_like(src)
    gpu.b.spinner_stream_copy(src, dst)
    t.cuda.synchronize()
    assert bool((src == dst).all())


def test_captured_graph_replays_match_eager(gpu, oracle):
    # the launch-bound small configuration is meant to be captured into a HIP graph: every replay, with eager
    # work and synchronisations in between, must give the bits of the eager call
    t, b = gpu.torch, gpu.b
    n, batch = 256, 1024
    x, d = _rng_case(n, batch, 4242)
    xt = _to(gpu, x)
    signs = b.spinner_pack_signs(_to(gpu, d[None]))
    eager = b.spinner_apply_signs(xt, signs, n, "none", 1.0)
    t.cuda.synchronize()
    want = oracle.apply(x, d[0], d[1], d[2], n, "none", 1.0)
    assert rel_l2_per_vector(eager.cpu().numpy(), want).max() <= REL_L2_TOL
    out = t.zeros_like(eager)
    side = t.cuda.Stream()
    side.wait_stream(t.cuda.current_stream())
    with t.cuda.stream(side):
        b.spinner_apply_signs(xt, signs, n, "none", 1.0, out=out)
    t.cuda.current_stream().wait_stream(side)
    t.cuda.synchronize()
    graph = t.cuda.CUDAGraph()
    with t.cuda.graph(graph):
        for _ in range(4):
            b.spinner_apply_signs(xt, signs, n, "none", 1.0, out=out)
    for rep in range(3):
        out.fill_(float(rep))                      # eager work between replays
        other = b.spinner_apply_signs(xt * 2.0, signs, n, "none", 1.0)
        t.cuda.synchronize()
        graph.replay()
        t.cuda.synchronize()
        assert t.equal(out, eager), rep
        assert t.equal(other, eager * 2.0)         # exact: a power-of-two factor commutes with every rounding


@pytest.mark.parametrize("n,m,L,epilogue,scale,batch", [(1024, 1024, 3, "none", 1.0, 21), (1024, 256, 4, "cossin", 32.0, 21),
                                                        (4096, 4096, 2, "cossin", 64.0, 9), (4096, 1000, 3, "none", 2.0, 9),
                                                        (1 << 15, 512, 2, "cossin", 8.0, 3), (1 << 17, 1 << 17, 2, "none", 1.0, 2),
                                                        (1 << 17, 1024, 3, "none", 4.0, 2)])
def test_stacked_blocks(gpu, oracle, n, m, L, epilogue, scale, batch):
    # Section 3.2: L independently drawn m-row blocks side by side (k = L m may exceed n)
    rng = np.random.default_rng(n + m + L)
    x = rng.standard_normal((batch, n)).astype(np.float32)
    if epilogue == "cossin":
        x *= np.float32(4.0 / math.sqrt(n))            # keeps w = scale * y at a few radians
    ds = W.rademacher_diagonals(n, 3 * L, 9000 + L + m).reshape(L, 3, n)
    got = gpu.b.spinner_apply_blocks(_to(gpu, x), _to(gpu, ds), m, epilogue, scale)
    gpu.torch.cuda.synchronize()
    got = got.cpu().numpy()
    want = oracle.apply_blocks(x, ds, m, epilogue, scale)
    assert got.shape == want.shape
    assert rel_l2_per_vector(got, want).max() <= REL_L2_TOL
    if L > 1 and n <= 4096:
        # block l of the stacked call is what the single-triple call gives for triple l (up to the 1/sqrt(L) of the features)
        # (the one-launch kernel orders its butterflies differently from the single-triple kernels: equal to rounding)
        one = _run_apply(gpu, x, ds[1], m, epilogue, scale)
        if epilogue == "none":
            assert rel_l2_per_vector(got[:, m:2 * m], one.astype(np.float64)).max() <= 2e-6
        else:
            assert np.allclose(got[:, m:2 * m] * math.sqrt(L), one[:, :m], rtol=1e-6, atol=1e-6)


@pytest.mark.parametrize("log2n", list(range(4, 15)))
def test_stacked_blocks_every_one_launch_size(gpu, oracle, log2n):
    # n <= 2^14: one kernel keeps x in registers and applies the L triples one after the other (features at 2^10 and 2^12: one
    # wave per block); both epilogues, all coordinates and a row limit that cuts through a tile (m a multiple of 4), batches
    # that leave part of a workgroup without a vector
    n = 1 << log2n
    batch = {4: 203, 5: 131, 6: 67}.get(log2n, 21 if log2n < 12 else 5)
    L = 3
    rng = np.random.default_rng(400 + log2n)
    x = rng.standard_normal((batch, n)).astype(np.float32)
    ds = W.rademacher_diagonals(n, 3 * L, 9100 + log2n).reshape(L, 3, n)
    ds[1, 2] = rng.standard_normal(n).astype(np.float32)          # a Gaussian third diagonal in one block
    xd, dsd = _to(gpu, x), _to(gpu, ds)
    for m in (n, max(4, (n // 2 + 4) & ~3), 4):
        got = gpu.b.spinner_apply_blocks(xd, dsd, m, "none", 1.5).cpu().numpy()
        want = oracle.apply_blocks(x, ds, m, "none", 1.5)
        assert got.shape == want.shape == (batch, L * m)
        for l in range(L):      # every block by itself: a block of few coordinates is not hidden behind the others
            err = rel_l2_first_m(got[:, l * m:(l + 1) * m], want[:, l * m:(l + 1) * m], x, n, m, 1.5)
            assert err.max() <= REL_L2_TOL, (log2n, m, l, err.max())
    xs = x * np.float32(4.0 / math.sqrt(n))
    xsd = _to(gpu, xs)
    for m in (n, max(4, (n // 4) & ~3)):
        scale = 0.5 * math.sqrt(n)
        got = gpu.b.spinner_apply_blocks(xsd, dsd, m, "cossin", scale).cpu().numpy()
        want = oracle.apply_blocks(xs, ds, m, "cossin", scale)
        assert got.shape == want.shape == (batch, 2 * L * m)
        assert rel_l2_per_vector(got, want).max() <= REL_L2_TOL, (log2n, m)


@pytest.mark.parametrize("n,m,L,batch", [(1 << 14, 1 << 14, 2, 256), (1 << 14, 4100, 3, 256),
                                             (1 << 12, 2560, 2, 256), (1 << 12, 4092, 2, 3072),
                                             (1 << 12, 4092, 3, 512), (1 << 12, 4092, 3, 1024)])
def test_stacked_features_on_both_sides_of_a_batch_limit(gpu, n, m, L, batch):
    # `batch` vectors and one more go to different kernels: fp64 butterflies in another order, so the features of the same
    # vectors agree to the rounding of their last two fp32 operations (a feature is at most 1 / sqrt(L m)), and the vector
    # that only the larger call has agrees with the single-triple calls
    t = gpu.torch
    g = t.Generator(device=gpu.dev)
    g.manual_seed(n + m + L)
    x = t.randn((batch + 1, n), generator=g, device=gpu.dev)
    ds = t.randint(0, 2, (L, 3, n), generator=g, device=gpu.dev).float() * 2.0 - 1.0
    below = gpu.b.spinner_apply_blocks(x[:batch], ds, m, "cossin", 64.0)
    above = gpu.b.spinner_apply_blocks(x, ds, m, "cossin", 64.0)
    tol = 2.0 ** -22 / math.sqrt(L * m)
    assert float((above[:batch] - below).abs().max()) <= tol
    for l in range(L):
        one = gpu.b.spinner_apply(x[batch:], ds[l, 0], ds[l, 1], ds[l, 2], m, "cossin", 64.0) / math.sqrt(L)
        both = t.cat((above[batch:, l * m:(l + 1) * m], above[batch:, (L + l) * m:(L + l + 1) * m]), 1)
        assert float((both - one).abs().max()) <= 2.0 * tol


@pytest.mark.parametrize("n,m,batch", [(1 << 13, 1 << 13, 256), (1 << 13, 501, 256), (1 << 13, 1 << 13, 768), (1 << 13, 501, 768),
                                       (1 << 14, 1 << 14, 256), (1 << 14, 8196, 256)])
def test_features_on_both_sides_of_a_batch_limit(gpu, n, m, batch):
    # `batch` vectors and one more go to kernels that differ in nothing but the registers they may take: the same bits
    t = gpu.torch
    g = t.Generator(device=gpu.dev)
    g.manual_seed(n + m)
    x = t.randn((batch + 1, n), generator=g, device=gpu.dev)
    d = t.randint(0, 2, (3, n), generator=g, device=gpu.dev).float() * 2.0 - 1.0
    words = gpu.b.spinner_pack_signs(d[None])
    for f in (lambda v: gpu.b.spinner_apply(v, d[0], d[1], d[2], m, "cossin", 64.0),
              lambda v: gpu.b.spinner_apply_signs(v, words, m, "cossin", 64.0)):
        assert t.equal(f(x)[:batch], f(x[:batch]))


@pytest.mark.parametrize("n", [16, 64, 256, 1024, 4096, 1 << 13, 1 << 14])
@pytest.mark.parametrize("L", [2, 5, 16])
def test_hash_of_few_vectors_cut_along_the_triples(gpu, n, L):
    # a launch of few waves applies the triples in several workgroups: the buckets of the same vectors in a batch that fills the
    # chip (4096 waves and five triples: one slice; 8192 waves and 16: four)
    t = gpu.torch
    batch = max(512, (1 << 22) // n)
    g = t.Generator(device=gpu.dev)
    g.manual_seed(n + L)
    x = t.randn((batch, n), generator=g, device=gpu.dev)
    d = t.randint(0, 2, (L, 3, n), generator=g, device=gpu.dev).float() * 2 - 1
    words = gpu.b.spinner_pack_signs(d)
    for call in (lambda v: gpu.b.spinner_hash(v, d), lambda v: gpu.b.spinner_hash_signs(v, words, L)):
        want = call(x)
        for few in (1, 19, 130):
            assert t.equal(call(x[:few]), want[:few]), few


@pytest.mark.parametrize("n,fills", [(64, 32768), (1024, 4096), (4096, 2048), (1 << 14, 512)])
@pytest.mark.parametrize("L", [3, 8, 13])
def test_hash_of_batches_that_fill_the_chip_once(gpu, n, fills, L):
    # one vector fewer, as many as and one more than give 4096 waves: slices of at least two, two and four triples, the last one
    # shorter; the buckets of a few vectors from the middle and both ends against those of the vectors alone
    t = gpu.torch
    g = t.Generator(device=gpu.dev)
    g.manual_seed(n + L)
    x = t.randn((fills + 1, n), generator=g, device=gpu.dev)
    d = t.randint(0, 2, (L, 3, n), generator=g, device=gpu.dev).float() * 2 - 1
    words = gpu.b.spinner_pack_signs(d)
    for call in (lambda v: gpu.b.spinner_hash(v, d), lambda v: gpu.b.spinner_hash_signs(v, words, L)):
        for batch in (fills - 1, fills, fills + 1):
            got = call(x[:batch])
            for part in (slice(0, 5), slice(fills // 2, fills // 2 + 5), slice(batch - 5, batch)):
                assert t.equal(got[part], call(x[:batch][part].contiguous())), batch


@pytest.mark.parametrize("epilogue", ["none", "cossin"])
@pytest.mark.parametrize("n, m", [(16, 16), (512, 512), (2048, 1000), (4096, 2560), (1 << 13, 1 << 13), (1 << 14, 4000)])
def test_stacked_blocks_of_few_vectors_cut_along_the_blocks(gpu, n, m, epilogue):
    # the same for stacked blocks: rows as in a batch of more than 2048 waves, which one workgroup takes through all blocks
    # (features of 2^14 from 257 vectors on run in another kernel with the same arithmetic)
    t, L = gpu.torch, 5
    batch = max(260, (1 << 24) // n)
    g = t.Generator(device=gpu.dev)
    g.manual_seed(n + m)
    x = t.randn((batch, n), generator=g, device=gpu.dev)
    d = t.randint(0, 2, (L, 3, n), generator=g, device=gpu.dev).float() * 2 - 1
    want = gpu.b.spinner_apply_blocks(x, d, m, epilogue, 1.5)
    for few in (1, 19, 130):
        got = gpu.b.spinner_apply_blocks(x[:few], d, m, epilogue, 1.5)
        # (other kernels serve some batches of features: sums in another order, a last place in the hardware's sine)
        assert float((got - want[:few]).abs().max()) <= (0.0 if epilogue == "none" else 1e-6 / (L * m) ** 0.5), few


def test_stacked_feature_blocks_in_slices(gpu):
    # n = 1024: one wave per pair of vectors and block, at most 2^24 workgroups per launch; with 2^18 blocks a launch takes
    # 128 vectors, so the last three rows of 131 come from a second one
    n, L, batch, m = 1024, 1 << 18, 131, 4
    g = gpu.torch.Generator(device=gpu.dev)
    g.manual_seed(9300)
    x = gpu.torch.randn((batch, n), generator=g, device=gpu.dev)
    ds = gpu.torch.randint(0, 2, (L, 3, n), generator=g, device=gpu.dev, dtype=gpu.torch.int8).to(gpu.torch.float32).mul_(2).sub_(1)
    got = gpu.b.spinner_apply_blocks(x, ds, m, "cossin", 32.0)
    assert gpu.torch.equal(got[120:], gpu.b.spinner_apply_blocks(x[120:].clone(), ds, m, "cossin", 32.0))
    one = gpu.b.spinner_apply(x, ds[L - 1, 0], ds[L - 1, 1], ds[L - 1, 2], m, "cossin", 32.0)
    last = gpu.torch.cat((got[:, (L - 1) * m:L * m], got[:, (2 * L - 1) * m:]), 1) * math.sqrt(L)
    assert gpu.torch.allclose(last, one, rtol=1e-6, atol=1e-6)


def test_stacked_blocks_errors(gpu):
    b, t = gpu.b, gpu.torch
    x = t.zeros((2, 256), dtype=t.float32, device=gpu.dev)
    ds = t.ones((2, 3, 256), dtype=t.float32, device=gpu.dev)
    with pytest.raises(b.SpinnerError) as e:
        b.spinner_apply_blocks(x, ds, 30, "none", 1.0)          # L > 1 needs m % 4 == 0
    assert e.value.status == b.SPINNER_ERR_BAD_M
    assert tuple(b.spinner_apply_blocks(x, ds[:1], 30, "none", 1.0).shape) == (2, 30)
    assert tuple(b.spinner_apply_blocks(x[:0], ds, 32, "cossin", 1.0).shape) == (0, 128)


# ------------------------------------------------------------------ seeded random shapes
def _random_cases(count, seed):
    rng = np.random.default_rng(seed)
    cases = []
    for _ in range(count):
        log2n = int(rng.integers(4, 15))
        n = 1 << log2n
        batch = int(rng.integers(1, 70 if log2n <= 11 else (20 if log2n <= 13 else 7)))
        kind = rng.integers(0, 4)
        if kind == 0:
            m = n
        elif kind == 1:
            m = int(rng.integers(1, n + 1))                        # any row limit, odd ones included
        elif kind == 2:
            m = max(1, n >> int(rng.integers(4, log2n + 1)))       # at or below n / 16: the pruned last round
        else:
            m = min(n, (n >> 4) + int(rng.integers(1, 9)))         # just above the pruning threshold
        cases.append((log2n, batch, m, ("none", "cossin")[int(rng.integers(0, 2))], ("fp32", "signs")[int(rng.integers(0, 2))],
                      int(rng.integers(0, 1 << 30))))
    return cases


@pytest.mark.parametrize("log2n,batch,m,epilogue,form,seed", _random_cases(36, 20261127))
def test_random_shapes_against_the_oracle(gpu, oracle, log2n, batch, m, epilogue, form, seed):
    n = 1 << log2n
    x, d = _rng_case(n, batch, seed)
    scale = 1.5 if epilogue == "none" else 2.0 * math.sqrt(n) / 8.0     # features: w of a few radians per unit of |x|
    if epilogue == "cossin":
        x *= np.float32(0.125)
    if form == "signs":
        signs = gpu.b.spinner_pack_signs(_to(gpu, d[None]))
        got = gpu.b.spinner_apply_signs(_to(gpu, x), signs, m, epilogue, scale).cpu().numpy()
    else:
        got = _run_apply(gpu, x, d, m, epilogue, scale)
    want = oracle.apply(x, d[0], d[1], d[2], m, epilogue, scale)
    assert got.shape == want.shape
    if epilogue == "none":
        # plain rule for m > 8; a handful of kept coordinates is measured against their expected size (helpers.py)
        assert rel_l2_first_m(got, want, x, n, m, scale).max() <= REL_L2_TOL, (log2n, batch, m, epilogue, form)
    else:
        assert rel_l2_per_vector(got, want).max() <= REL_L2_TOL, (log2n, batch, m, epilogue, form)
