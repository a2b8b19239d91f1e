"""Float32 layers at the ends of the number range, where operands split into bfloat16 terms need care: the results are those of float32
arithmetic, forward, both gradients, in one part and in several."""
import numpy as np
import pytest

from paper_1909_09577_amd import binding as nm

pytestmark = pytest.mark.gpu

# B, Cin, Cout, T, K: one part; few tiles, whose reduction channels are shared; 13 taps
DIMS = [(9, 64, 96, 200, 11), (1, 200, 72, 77, 11), (3, 130, 40, 60, 13)]


def _calls(dims, x, w, dy, **more):
    import torch
    B, Cin, Cout, T, K = dims
    kw = dict(stride=1, dilation=1, pad=K // 2, relu=False, **more)
    xd, wd, dyd = (torch.from_numpy(np.asarray(a, dtype=np.float32)).cuda() for a in (x, w, dy))
    y = nm.nm_conv1d_block_fwd(xd, wd, None, None, None, **kw)
    dx, _ = nm.nm_conv1d_bwd_data(dyd, wd, T, **kw)
    dw = nm.nm_conv1d_bwd_weight(xd, dyd, K, **kw)
    return [t.cpu().numpy() for t in (y, dx, dw)]


@pytest.mark.parametrize("dims", DIMS, ids=str)
def test_products_at_the_top_of_the_range(dims):
    """Single products of 2^64*(1 - 2^-10) twice, 3.396e38: finite, although both operands round up to 2^64 as bfloat16 values.  A sum of
    one product is correctly rounded in float32; 2^-22 allows for what a split drops (below 2^-25)."""
    B, Cin, Cout, T, K = dims
    big = np.float32(2.0 ** 64 * (1 - 2.0 ** -10))
    x, w, dy = np.zeros((B, Cin, T)), np.zeros((Cout, Cin, K)), np.zeros((B, Cout, T))
    x[:, 3, T // 2], w[:, 3, K // 2], dy[:, 5, T // 2] = big, big, -big
    y, dx, dw = _calls(dims, x, w, dy)
    want = float(big) ** 2
    near = lambda got, ref: abs(float(got) / ref - 1) < 2.0 ** -22
    assert all(near(v, want) for v in y[:, :, T // 2].ravel())
    assert all(near(v, -want) for v in dx[:, 3, T // 2].ravel())
    # B products, minus 3.396e38 each: one is finite, more are infinite
    assert near(dw[5, 3, K // 2], -want) if B == 1 else dw[5, 3, K // 2] == -np.inf
    for t in (y, dx):
        assert np.isfinite(t).all()


@pytest.mark.parametrize("dims", DIMS, ids=str)
def test_infinities_and_overflow(dims):
    """Sums that overflow, and infinite operands, are what the plain kernels make of them."""
    rng = np.random.default_rng(1)
    B, Cin, Cout, T, K = dims
    x, w, dy = rng.standard_normal((B, Cin, T)), rng.standard_normal((Cout, Cin, K)), rng.standard_normal((B, Cout, T))
    x[0, 1, 7], w[2, 2, 0], dy[0, 3, 9] = np.inf, -np.inf, np.inf
    x[B - 1, 4, T - 3] = w[7, 4, 1] = dy[B - 1, 7, T - 3] = 3e38
    for got, ref in zip(_calls(dims, x, w, dy), _calls(dims, x, w, dy, force_direct=True)):
        assert not np.isfinite(ref).all() and np.isfinite(ref).any()
        fin = np.isfinite(ref)
        assert np.array_equal(np.isfinite(got), fin) and np.array_equal(got[~fin], ref[~fin], equal_nan=True)
        # (rows with a finite 3e38 in them have finite results of that size: scaled by each channel's largest)
        top = np.abs(np.where(fin, ref, 0)).max()
        assert np.abs(np.where(fin, got, 0) - np.where(fin, ref, 0)).max() <= 1e-5 * top


# sizes of the two operands of a pass: float32's smallest normal numbers, denormal ones, the edges of what bfloat16 terms hold as they are
SIZES = [(-126, 100), (-140, 120), (-109, 90), (-115, 20), (110, -100), (120, -126), (-70, -60)]


@pytest.mark.parametrize("swap", [False, True], ids=["", "swapped"])
@pytest.mark.parametrize("sizes", SIZES, ids=str)
def test_operands_of_any_size(sizes, swap):
    """The error stays that of float32 sums (1e-6 of the result, 2e-7 being measured) wherever the results are normal numbers; of
    results below 2^-126 it stays below the sum of their roundings, half of 2^-149 for each of a few hundred products."""
    import torch
    from oracle import conv1d_oracle as orc
    a, b = (2.0 ** e for e in (sizes[::-1] if swap else sizes))
    rng = np.random.default_rng(4)
    B, C, M, T, K = 2, 64, 48, 70, 11
    kw = dict(stride=1, dilation=1, pad=5)
    draw = lambda size, *s: (rng.standard_normal(s) * size).astype(np.float32)
    dev = lambda v: torch.from_numpy(v).cuda()
    x, dy, w_x, w_dy, dy_x = draw(a, B, C, T), draw(a, B, M, T), draw(b, M, C, K), draw(b, M, C, K), draw(b, B, M, T)
    for got, ref in ((nm.nm_conv1d_block_fwd(dev(x), dev(w_x), None, None, None, relu=False, **kw), orc.block_fwd(x, w_x, None, None, None, False, **kw)),
                     (nm.nm_conv1d_bwd_data(dev(dy), dev(w_dy), T, relu=False, **kw)[0], orc.bwd_data(dy, w_dy, T, **kw)),
                     (nm.nm_conv1d_bwd_weight(dev(x), dev(dy_x), K, relu=False, **kw), orc.bwd_weight(x, dy_x, K, **kw))):
        ref = np.asarray(ref, dtype=np.float64)
        assert np.isfinite(ref).all() and np.linalg.norm(ref) > 0
        off = np.linalg.norm(got.double().cpu().numpy() - ref)
        assert off <= 1e-6 * np.linalg.norm(ref) + (2.0 ** -149 * 500 * ref.size ** 0.5 if sum(sizes) < -100 else 0), (off / np.linalg.norm(ref))
