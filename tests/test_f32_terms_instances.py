"""Every instance of the float32 kernels on bfloat16 terms: which one a geometry runs on, with how many parts (host only, from the launches
themselves), and its results on the device, also where a wavefront's sums are as long as they may be and one step longer."""
import pytest

import _launches as la
import test_gpu_f32 as base
from paper_1909_09577_amd import binding as nm

# (tile in 32 steps, gradient, taps, in parts): B, Cin, Cout, T
CONVS = {
    (1, 0, 11, 0): (2, 20, 32, 37), (1, 0, 11, 1): (2, 69, 27, 29), (1, 0, 13, 0): (2, 22, 16, 84), (1, 0, 13, 1): (1, 109, 34, 44),
    (1, 1, 11, 0): (2, 20, 32, 37), (1, 1, 11, 1): (1, 31, 145, 46), (1, 1, 13, 0): (2, 22, 16, 84), (1, 1, 13, 1): (7, 21, 67, 26),
    (2, 0, 11, 0): (13, 17, 33, 458), (2, 0, 11, 1): (8, 146, 48, 176), (2, 0, 13, 0): (19, 19, 159, 66), (2, 0, 13, 1): (3, 135, 34, 506),
    (2, 1, 11, 0): (20, 76, 19, 134), (2, 1, 11, 1): (15, 65, 236, 36), (2, 1, 13, 0): (23, 99, 17, 79), (2, 1, 13, 1): (4, 38, 153, 340),
    (3, 0, 11, 0): (15, 16, 208, 129), (3, 0, 11, 1): (5, 327, 33, 522), (3, 0, 13, 0): (19, 20, 247, 67), (3, 0, 13, 1): (17, 270, 40, 151),
    (3, 1, 11, 0): (23, 115, 17, 168), (3, 1, 11, 1): (23, 37, 338, 93), (3, 1, 13, 0): (15, 33, 27, 567), (3, 1, 13, 1): (24, 46, 350, 70),
}
# a wavefront's taps: B, Cin, Cout, T, K (odd, even, three groups of taps)
WGRADS = {2: (2, 40, 48, 65, 3), 4: (3, 31, 33, 129, 8), 6: (4, 70, 131, 193, 31)}
# 42 links of a chain, the most that run on terms, and the next longer ones; tiles too many to share, so that no part shortens a chain
LINKS = {(26, 384, 20, 150, 13): True, (26, 392, 20, 150, 13): False, (26, 448, 20, 150, 11): True, (26, 449, 20, 150, 11): False}
FLIPPED = {(B, M, R, T, K): there for (B, R, M, T, K), there in LINKS.items()}


def _dims(B, Cin, Cout, T, K):
    return (B, Cin, Cout, T, K, 1, 1, K // 2)


def _kernels(calls):
    """Main kernels of the calls: (name, template arguments) and grid."""
    out = []
    for status, seq in la.run(calls, instances=True):
        assert status == nm.NM_OK
        out.append(next((what, grid) for _, what, grid in seq if what[0] in ("f32_conv_kernel", "f32_wgrad_kernel")))
    return out


def test_every_convolution_instance_has_a_case():
    assert set(CONVS) == {(nt, flip, k, split) for nt in (1, 2, 3) for flip in (0, 1) for k in (11, 13) for split in (0, 1)}
    got = _kernels([{"call": "bwd_data" if key[1] else "fwd", "dims": _dims(*d, key[2]), "dtype": nm.NM_F32} for key, d in CONVS.items()])
    for key, (what, grid) in zip(CONVS, got):
        assert what == ("f32_conv_kernel", *key) and (grid[1] > 1) == bool(key[3]), (key, what, grid)


def test_weight_gradient_instances():
    got = _kernels([{"call": "bwd_weight", "dims": _dims(*d), "dtype": nm.NM_F32} for d in WGRADS.values()])
    assert [what for what, _ in got] == [("f32_wgrad_kernel", taps) for taps in WGRADS]


@pytest.mark.parametrize("size,parts", [((6, 384, 384, 100, 13), [1, 2]), ((16, 256, 256, 304, 29), [1, 1, 1, 4])], ids=str)
def test_parts_of_a_weight_gradient_within_the_room(size, parts):
    """The number that is estimated to be fastest of those that fit, told by the workgroups; a byte less than a part needs is no room for it."""
    B, Cin, Cout, T, K = size
    g, part, tiles = 4 * B * Cout * T, 4 * Cin * Cout * K, -(-Cin // 32) * -(-Cout // 32) * -(-K // 12)
    assert g % 256 == part % 256 == 0 and nm.nm_conv1d_workspace_bytes(nm.NM_OP_BWD_WEIGHT, *_dims(*size), nm.NM_F32, 0) == g + len(parts) * part
    rooms = [(s, g + n * part) for n, s in enumerate(parts, 1)] + [(s, g + n * part - 1) for n, s in enumerate(parts[:-1], 2)]
    got = _kernels([{"call": "bwd_weight", "dims": _dims(*size), "dtype": nm.NM_F32, "ws_bytes": room} for _, room in rooms])
    for (s, room), (what, grid) in zip(rooms, got):
        assert what[0] == "f32_wgrad_kernel" and len(what) == 2 and grid[0] == tiles * s, (s, room, what, grid)


def test_links():
    for op, table in (("fwd", LINKS), ("bwd_data", FLIPPED)):
        got = _kernels([{"call": op, "dims": _dims(*d), "dtype": nm.NM_F32} for d in table])
        for (d, there), (what, grid) in zip(table.items(), got):
            assert (len(what) == 5) == there and grid[1] == 1, (d, what, grid)  # (the other engine's instances have five arguments)


def _layer(i, B, Cin, Cout, T, K):
    return base.L("x".join(map(str, (B, Cin, Cout, T, K))), B, Cin, Cout, T, K, pad=K // 2, residual=i % 2 == 0, relu=i % 3 > 0)


SIZES = list(dict.fromkeys([(*d, key[2]) for key, d in CONVS.items()] + list(WGRADS.values()) + list(LINKS) + list(FLIPPED)))


@pytest.mark.gpu
@pytest.mark.parametrize("masked", [False, True], ids=["full", "lengths"])
@pytest.mark.parametrize("cfg", [_layer(i, *d) for i, d in enumerate(SIZES)], ids=lambda c: c.name)
def test_results(cfg, masked):
    """The other float32 layers' gates: 1e-5 of the result, no less exact than the plain kernels."""
    base.test_float32_on_the_matrix_cores(cfg, masked)


@pytest.mark.gpu
@pytest.mark.parametrize("B,Cin,Cout,T,K", [(32, 64, 96, 800, 5), (16, 128, 128, 1600, 3), (32, 64, 64, 800, 11), (1, 96, 64, 20000, 13),
                                            (300, 32, 64, 70, 3), (500, 32, 64, 16, 5)])
def test_long_sums_of_a_weight_gradient(B, Cin, Cout, T, K):
    """No rounding goes one way: the mean error, over some thousand elements, is a small part of the error, which is that of n additions of random
    terms to their own sum, about 0.58 * 2^-24 * sqrt(n / 2): 2.1e-7 for the 75 units of a part that the largest of these has, plus a little for
    the parts and slices.  (The matrix instructions cut downwards: mean -3.4e-7, 3.7e-7 in all in the first three before the signs took turns.)"""
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(7)
    x, dy = (torch.randn(B, c, T, device="cuda", generator=g) for c in (Cin, Cout))
    dw = nm.nm_conv1d_bwd_weight(x, dy, K, stride=1, dilation=1, pad=K // 2, relu=False)
    xp = torch.nn.functional.pad(x.double(), (K // 2, K // 2))
    rows = dy.double().transpose(0, 1).reshape(Cout, -1)
    ref = torch.stack([rows @ xp[:, :, k:k + T].transpose(1, 2).reshape(-1, Cin) for k in range(K)], 2)
    off, size = dw.double() - ref, ref.pow(2).mean().sqrt()
    assert float(off.mean().abs() / size) <= 2e-8 and float(off.pow(2).mean().sqrt() / size) <= 2.5e-7
