"""GPU parity of the adaptive layer (learned diagonals): forward with saved activations and backward pass,
called through the C ABI, against the fp64 oracle on the same fp32 inputs.

Tolerance: relative L2 error <= 1e-5 per vector for y and dx, and per diagonal for the three parameter
gradients (which sum over the batch)."""
import math
import sys

import numpy as np
import pytest

from helpers import REL_L2_TOL, rel_l2_per_vector

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


def _to(g, a):
    return g.torch.from_numpy(np.ascontiguousarray(a)).to(g.dev)


def _case(n, batch, seed):
    rng = np.random.default_rng(seed)
    x = rng.standard_normal((batch, n)).astype(np.float32)
    d = (rng.standard_normal((3, n)) * 0.5 + 1.0).astype(np.float32)       # learned diagonals: arbitrary reals
    dy = rng.standard_normal((batch, n)).astype(np.float32)
    return x, d, dy


def _run(g, x, d, dy, scale):
    xt, dt, dyt = _to(g, x), _to(g, d), _to(g, dy)
    y, saved = g.b.spinner_layer_forward(xt, dt[0], dt[1], dt[2], scale)
    dx, dd = g.b.spinner_layer_backward(dyt, xt, saved, dt[0], dt[1], dt[2], scale)
    g.torch.cuda.synchronize()
    return y.cpu().numpy(), dx.cpu().numpy(), dd.cpu().numpy()


def _check(oracle, x, d, dy, scale, y, dx, dd):
    wy, _, _ = oracle.layer_forward(x, d[0], d[1], d[2], scale)
    wdx, wdd = oracle.layer_backward(x, d[0], d[1], d[2], dy, scale)
    assert rel_l2_per_vector(y, wy).max() <= REL_L2_TOL
    assert rel_l2_per_vector(dx, wdx).max() <= REL_L2_TOL
    err = rel_l2_per_vector(dd, wdd)
    assert err.max() <= REL_L2_TOL, err


@pytest.mark.parametrize("log2n", list(range(4, 15)))
def test_layer_forward_backward_every_size(gpu, oracle, log2n):
    n = 1 << log2n
    batch = {4: 1000, 5: 777, 6: 333, 7: 200, 13: 7, 14: 5}.get(log2n, 37 if log2n < 12 else 9)
    x, d, dy = _case(n, batch, 6000 + log2n)
    scale = 1.0 if log2n % 2 else 0.37
    y, dx, dd = _run(gpu, x, d, dy, scale)
    _check(oracle, x, d, dy, scale, y, dx, dd)


@pytest.mark.parametrize("log2n,batch", [(15, 5), (16, 3), (17, 70), (19, 2), (20, 2)])
def test_layer_above_the_fused_range(gpu, oracle, log2n, batch):
    # single transforms as a pass over rows and a pass over columns, the signals of the backward pass materialised,
    # the diagonal gradients as batch sums; (17, 70): more vectors than slabs of the batch sum
    n = 1 << log2n
    x, d, dy = _case(n, batch, 6300 + log2n)
    scale = 1.0 if log2n % 2 else 1.7
    y, dx, dd = _run(gpu, x, d, dy, scale)
    _check(oracle, x, d, dy, scale, y, dx, dd)
    # dx written over dy; the forward pass agrees with the projection entry point
    xt, dt, dyt = _to(gpu, x), _to(gpu, d), _to(gpu, dy)
    y1, saved = gpu.b.spinner_layer_forward(xt, dt[0], dt[1], dt[2], scale)
    dx2, dd2 = gpu.b.spinner_layer_backward(dyt, xt, saved, dt[0], dt[1], dt[2], scale, dx=dyt)
    y3 = gpu.b.spinner_apply(xt, dt[0], dt[1], dt[2], n, "none", scale)
    gpu.torch.cuda.synchronize()
    assert dx2.data_ptr() == dyt.data_ptr()
    assert np.array_equal(dx2.cpu().numpy(), dx) and np.array_equal(dd2.cpu().numpy(), dd)
    assert rel_l2_per_vector(y1.cpu().numpy(), y3.cpu().numpy().astype(np.float64)).max() <= 2e-6


@pytest.mark.parametrize("n,batch", [(1 << 15, 33), (1 << 15, 300), (1 << 16, 49)])
def test_layer_of_the_widest_sizes_on_both_sides_of_the_batch_limit(gpu, n, batch):
    # more than 32 (2^16: 48) vectors go through one kernel per pass, fewer through global memory; what the one saves the other
    # reads: the forward pass of the whole batch, then backward passes of the whole and of its first five vectors
    t, b = gpu.torch, gpu.b
    g = t.Generator(device=gpu.dev)
    g.manual_seed(n + batch)
    x, dy = (t.randn((batch, n), generator=g, device=gpu.dev) for _ in range(2))
    d = 1.0 + 0.5 * t.randn((3, n), generator=g, device=gpu.dev)
    y, saved = b.spinner_layer_forward(x, d[0], d[1], d[2], 0.8)
    dx, dd = b.spinner_layer_backward(dy, x, saved, d[0], d[1], d[2], 0.8)
    few = b.spinner_layer_forward(x[:5], d[0], d[1], d[2], 0.8)
    # fp32 rounding of 3 log2(n) stages in two orders
    assert float((few[0] - y[:5]).norm() / y[:5].norm()) <= 1e-6
    part = saved.view(2, batch, n)[:, :5].contiguous()
    assert float((few[1] - part).norm() / part.norm()) <= 1e-6
    a = b.spinner_layer_backward(dy[:5], x[:5], part, d[0], d[1], d[2], 0.8)
    assert float((a[0] - dx[:5]).norm() / dx[:5].norm()) <= 1e-6
    rest = saved.view(2, batch, n)[:, 5:].contiguous()
    c = b.spinner_layer_backward(dy[5:], x[5:], rest, d[0], d[1], d[2], 0.8)
    assert float(((a[1].double() + c[1].double() - dd.double()).norm(dim=1) / dd.double().norm(dim=1)).max()) <= 2e-6
    inner = float((dy.double() * y.double()).sum())
    for k in range(3):
        assert abs(float((d[k].double() * dd[k].double()).sum()) - inner) <= 1e-5 * abs(inner) + 1e-2
    over = dy.clone()
    dx2, dd2 = b.spinner_layer_backward(over, x, saved, d[0], d[1], d[2], 0.8, dx=over)
    assert t.equal(dx2, dx) and t.equal(dd2, dd)


@pytest.mark.parametrize("n,batch", [(1 << 15, 32), (1 << 15, 33), (1 << 16, 48), (1 << 16, 49)])
def test_layer_of_the_widest_sizes_over_the_range_of_fp32(gpu, n, batch):
    # on both sides of the batch limit the values are normalised on the way: inputs and scales times powers of two, up to where a
    # transform's own sums come near 2^128, give the same bits times that power (but for the roundings of denormal numbers, which none
    # of these has); the scale's power counts from the first transform of the backward pass on
    t, b = gpu.torch, gpu.b
    g = t.Generator(device=gpu.dev)
    g.manual_seed(n + batch)
    x, dy = (t.randn((batch, n), generator=g, device=gpu.dev) for _ in range(2))
    d = t.randint(0, 2, (3, n), generator=g, device=gpu.dev).float() * 2 - 1

    def step(x, dy, scale, scale_back):
        y, saved = b.spinner_layer_forward(x, d[0], d[1], d[2], scale)
        dx, dd = b.spinner_layer_backward(dy, x, saved, d[0], d[1], d[2], scale_back)
        return y, saved, dx, dd

    want = step(x, dy, 0.75, 0.75)
    assert all(bool(t.isfinite(r).all()) for r in want)
    # powers of x, dy, the forward and the backward scale
    for px, pd, ps, pb in ((110, 0, 0, 0), (0, 110, 0, 0), (-60, 0, 0, 0), (0, -60, 0, 0), (60, -60, 0, 0), (0, 0, 120, 100), (0, 0, -90, -60),
                           (100, 0, -100, -60), (60, 110, 0, -110)):
        y, saved, dx, dd = step(x * 2.0 ** px, dy * 2.0 ** pd, 0.75 * 2.0 ** ps, 0.75 * 2.0 ** pb)
        what = (px, pd, ps, pb)
        if px + ps <= 120:
            assert t.equal(y, want[0] * 2.0 ** (px + ps)), what
        assert t.equal(saved, want[1] * 2.0 ** px), what
        assert t.equal(dx, want[2] * 2.0 ** (pd + pb)), what
        assert t.equal(dd, want[3] * 2.0 ** (px + pd + pb)), what


def test_layer_above_the_fused_range_in_several_slices(gpu):
    # n = 2^17: the passes walk the batch in slices of 512 vectors; 513 vectors leave a second, shorter slice (257 + 256).
    # Vectors are independent, so y and dx of any row must have the bits of a run on that row alone; each diagonal
    # gradient satisfies sum_i d_k[i] dd_k[i] = <dy, y> (the layer is linear in each diagonal).
    t = gpu.torch
    n, batch = 1 << 17, 513
    g = t.Generator(device=gpu.dev)
    g.manual_seed(6400)
    x = t.randn((batch, n), generator=g, device=gpu.dev, dtype=t.float32)
    dy = t.randn((batch, n), generator=g, device=gpu.dev, dtype=t.float32)
    d = t.randn((3, n), generator=g, device=gpu.dev, dtype=t.float32) * 0.5 + 1.0
    y, saved = gpu.b.spinner_layer_forward(x, d[0], d[1], d[2], 1.3)
    dx, dd = gpu.b.spinner_layer_backward(dy, x, saved, d[0], d[1], d[2], 1.3)
    rows = [0, 255, 256, 257, 511, 512]
    xs, dys = x[rows].contiguous(), dy[rows].contiguous()
    ys, saved_s = gpu.b.spinner_layer_forward(xs, d[0], d[1], d[2], 1.3)
    dxs, _ = gpu.b.spinner_layer_backward(dys, xs, saved_s, d[0], d[1], d[2], 1.3)
    t.cuda.synchronize()
    assert t.equal(y[rows], ys) and t.equal(dx[rows], dxs)
    inner = float((dy.double() * y.double()).sum())
    for k in range(3):
        assert abs(float((d[k].double() * dd[k].double()).sum()) - inner) <= 1e-5 * abs(inner)


@pytest.mark.parametrize("n,batch", [(64, 70000), (256, 20000), (2048, 2300), (4096, 1100), (8192, 700), (16384, 600)])
def test_layer_backward_many_vectors_per_slot(gpu, oracle, n, batch):
    # more vectors than resident tile slots: every slot accumulates several vectors, the last round is ragged
    x, d, dy = _case(n, batch, 6100 + n)
    assert gpu.b.spinner_layer_workspace_bytes(n, batch) < batch * 3 * n * 4
    y, dx, dd = _run(gpu, x, d, dy, 1.0)
    _check(oracle, x, d, dy, 1.0, y, dx, dd)


@pytest.mark.parametrize("n,batch", [(16, 1), (16, 65), (16, 98305), (32, 33), (32, 50001), (64, 8000), (128, 17), (256, 8193), (512, 5),
                                     (512, 4097), (1024, 3), (1024, 4099), (2048, 33), (8192, 20)])
def test_layer_diagonal_gradients_of_whole_workgroups(gpu, n, batch):
    # up to n = 1024 a workgroup adds up its tiles in fp64 and writes one row (edges: a workgroup that is not full, one vector more
    # than all workgroups hold at once), above it writes a row per tile and few rows are added by smaller blocks: the gradients
    # against fp64 matrix products, and nothing written past the documented workspace
    t, b = gpu.torch, gpu.b
    g = t.Generator(device=gpu.dev)
    g.manual_seed(n + batch)
    x, dy = (t.randn((batch, n), generator=g, device=gpu.dev) for _ in range(2))
    d = 1.0 + 0.5 * t.randn((3, n), generator=g, device=gpu.dev)
    _, saved = b.spinner_layer_forward(x, d[0], d[1], d[2])
    need = b.spinner_layer_workspace_bytes(n, batch)
    ws = t.full((need + 4096,), 0xA5, dtype=t.uint8, device=gpu.dev)
    dx, dd = b.spinner_layer_backward(dy, x, saved, d[0], d[1], d[2], workspace=ws)
    assert bool((ws[need:] == 0xA5).all())
    H = t.ones((1, 1), dtype=t.float64, device=gpu.dev)
    while H.shape[0] < n:
        H = t.cat((t.cat((H, H), 1), t.cat((H, -H), 1)), 0)
    H /= math.sqrt(n)
    a, D = [x.double()], d.double()
    for k in range(2):
        a.append((a[-1] * D[k]) @ H)
    s, want = dy.double() @ H, [None] * 3
    for k in (2, 1, 0):
        want[k] = (s * a[k]).sum(0)
        s = (s * D[k]) @ H if k else s * D[0]
    want = t.stack(want)
    # 3 log2(n) rounded stages per factor of a product (2^-24 each, independent) leave some 4e-7 of the norm at n = 2^13
    assert float(((dd.double() - want).norm(dim=1) / want.norm(dim=1)).max()) <= 1.5e-6
    assert float((dx.double() - s).norm() / s.norm()) <= 1.5e-6


@pytest.mark.parametrize("n", [16, 256, 2048, 1 << 14])
def test_layer_of_large_batches(gpu, n):
    # from 2^24 elements on the backward kernels carry the non-temporal hint: the same bits per vector as for a small batch, and
    # diagonal gradients that are the sum of those of parts below the limit (fp32 running sums over at most batch / 8192 ..
    # batch / 512 vectors per slot, slots added in fp64: 1e-6 of the norm leaves a factor of five)
    t = gpu.torch
    batch = (1 << 25) // n + 3
    g = t.Generator(device=gpu.dev)
    g.manual_seed(n)
    x = t.randn((batch, n), generator=g, device=gpu.dev)
    dy = t.randn((batch, n), generator=g, device=gpu.dev)
    d = 1.0 + 0.5 * t.randn((3, n), generator=g, device=gpu.dev)

    def step(r):
        y, saved = gpu.b.spinner_layer_forward(x[r], d[0], d[1], d[2], 0.75)
        return (y, *gpu.b.spinner_layer_backward(dy[r], x[r], saved, d[0], d[1], d[2], 0.75))

    y, dx, dd = step(slice(0, batch))
    parts = [step(slice(i, min(batch, i + (1 << 23) // n))) for i in range(0, batch, (1 << 23) // n)]
    assert t.equal(y, t.cat([p[0] for p in parts])) and t.equal(dx, t.cat([p[1] for p in parts]))
    want = sum(p[2].double() for p in parts)
    assert float((dd.double() - want).norm() / want.norm()) <= 1e-6


def test_layer_special_cases(gpu, oracle):
    n, batch = 1024, 19
    x, d, dy = _case(n, batch, 6200)
    ones = np.ones((3, n), dtype=np.float32)
    # identity diagonals: y = H x, dx = H dy, and all three parameter gradients equal sum_b (H dy) * (H^k x) terms
    y, dx, dd = _run(gpu, x, ones, dy, 1.0)
    _check(oracle, x, ones, dy, 1.0, y, dx, dd)
    # forward agrees with the projection entry point on the same inputs
    xt, dt = _to(gpu, x), _to(gpu, d)
    y2, _ = gpu.b.spinner_layer_forward(xt, dt[0], dt[1], dt[2], 2.0)
    y3 = gpu.b.spinner_apply(xt, dt[0], dt[1], dt[2], n, "none", 2.0)
    gpu.torch.cuda.synchronize()
    assert rel_l2_per_vector(y2.cpu().numpy(), y3.cpu().numpy().astype(np.float64)).max() <= 1e-6
    # dx written over dy; two runs give identical bits (no atomics anywhere)
    dyt = _to(gpu, dy)
    _, saved = gpu.b.spinner_layer_forward(xt, dt[0], dt[1], dt[2], 1.0)
    dx1, dd1 = gpu.b.spinner_layer_backward(dyt, xt, saved, dt[0], dt[1], dt[2], 1.0)
    dx2, dd2 = gpu.b.spinner_layer_backward(dyt, xt, saved, dt[0], dt[1], dt[2], 1.0, dx=dyt)
    gpu.torch.cuda.synchronize()
    assert gpu.torch.equal(dx1, dx2) and gpu.torch.equal(dd1, dd2) and dx2.data_ptr() == dyt.data_ptr()
    # the layer is linear in each diagonal: sum_i d_k[i] dd_k[i] = <dy, y>
    y1, _, dd3 = _run(gpu, x, d, dy, 1.0)
    inner = float((dy.astype(np.float64) * y1).sum())
    for k in range(3):
        assert abs(float((d[k].astype(np.float64) * dd3[k]).sum()) - inner) <= 1e-4 * abs(inner) + 1e-3


def test_layer_empty_batch_and_errors(gpu):
    b, t = gpu.b, gpu.torch
    d = t.ones(256, dtype=t.float32, device=gpu.dev)
    x = t.zeros((0, 256), dtype=t.float32, device=gpu.dev)
    y, saved = b.spinner_layer_forward(x, d, d, d)
    assert tuple(y.shape) == (0, 256)
    bad = t.zeros((2, 1000), dtype=t.float32, device=gpu.dev)
    dbad = t.ones(1000, dtype=t.float32, device=gpu.dev)
    with pytest.raises(b.SpinnerError) as e:
        b.spinner_layer_forward(bad, dbad, dbad, dbad)
    assert e.value.status == b.SPINNER_ERR_BAD_N


def test_layer_step_as_a_captured_graph(gpu):
    # a training step at the small hidden sizes is launch-bound and meant to be captured: every replay, with
    # eager work and synchronisations in between, must give the bits of the eager forward + backward calls
    t, b = gpu.torch, gpu.b
    n, batch = 256, 1024
    x, d, dy = _case(n, batch, 777)
    xt, dt, dyt = _to(gpu, x), _to(gpu, d), _to(gpu, dy)
    y0, saved0 = b.spinner_layer_forward(xt, dt[0], dt[1], dt[2], 1.0)
    dx0, dd0 = b.spinner_layer_backward(dyt, xt, saved0, dt[0], dt[1], dt[2], 1.0)
    t.cuda.synchronize()
    y, saved, dx, dd = t.zeros_like(y0), t.zeros_like(saved0), t.zeros_like(dx0), t.zeros_like(dd0)
    ws = t.empty(max(16, b.spinner_layer_workspace_bytes(n, batch)), dtype=t.uint8, device=gpu.dev)

    def step():
        b.spinner_layer_forward(xt, dt[0], dt[1], dt[2], 1.0, y=y, saved=saved)
        b.spinner_layer_backward(dyt, xt, saved, dt[0], dt[1], dt[2], 1.0, dx=dx, dd=dd, workspace=ws)

    side = t.cuda.Stream()
    side.wait_stream(t.cuda.current_stream())
    with t.cuda.stream(side):
        step()
    t.cuda.current_stream().wait_stream(side)
    t.cuda.synchronize()
    graph = t.cuda.CUDAGraph()
    with t.cuda.graph(graph):
        for _ in range(3):
            step()
    for rep in range(3):
        for buf in (y, saved, dx, dd):
            buf.fill_(float(rep))                  # eager work between replays
        ws.zero_()
        t.cuda.synchronize()
        graph.replay()
        t.cuda.synchronize()
        assert t.equal(y, y0) and t.equal(dx, dx0) and t.equal(dd, dd0), rep
