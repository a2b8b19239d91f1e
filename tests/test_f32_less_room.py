"""Float32 weight gradients with room for fewer parts than are asked for, but for those of the kernel on the float32 instructions (what was
asked for when it was the only one): they stay on the matrix cores, with no more parts than fit.  Without room for any the plain kernel runs."""
import numpy as np
import pytest

from paper_1909_09577_amd import binding as nm

# dims, rooms of the weight gradient alone and of both gradients
CASES = [((6, 384, 384, 100, 13, 1, 1, 6), 8589312, 9510912), ((2, 384, 256, 304, 25, 1, 1, 12), 10452992, 12943360),
         ((16, 256, 256, 304, 29, 1, 1, 14), 25165824, None)]


@pytest.mark.parametrize("dims,room,_", CASES, ids=lambda v: str(v))
def test_kernel(dims, room, _):
    asked = nm.nm_conv1d_workspace_bytes(nm.NM_OP_BWD_WEIGHT, *dims, nm.NM_F32, 1)
    part = 4 * dims[1] * dims[2] * dims[4]
    assert room + part <= asked
    for n, name in ((asked, "f32_wgrad_kernel"), (room, "f32_wgrad_kernel"), (4 * dims[0] * dims[2] * dims[3], "direct")):
        assert nm.nm_conv1d_kernel_name(nm.NM_OP_BWD_WEIGHT, *dims, dtype=nm.NM_F32, flags=1, workspace_bytes=n).startswith(name)


@pytest.mark.gpu
@pytest.mark.parametrize("dims,room,both", CASES[:2], ids=lambda v: str(v))
def test_results(dims, room, both):
    """The bytes behind the room stay as they are; the gate is that of the other float32 tests, 1e-5 of the result."""
    import torch
    from oracle import conv1d_oracle as orc
    B, Cin, Cout, T, K, _, _, pad = dims
    rng = np.random.default_rng(5)
    x, dy = rng.standard_normal((B, Cin, T)).astype(np.float32), rng.standard_normal((B, Cout, T)).astype(np.float32)
    w = (rng.standard_normal((Cout, Cin, K)) / (Cin * K) ** 0.5).astype(np.float32)
    kw = dict(stride=1, dilation=1, pad=pad)
    ref_dw, ref_dx = orc.bwd_weight(x, dy, K, **kw), orc.bwd_data(dy, w, T, **kw)
    xd, dyd, wd = (torch.from_numpy(a).cuda() for a in (x, dy, w))

    def near(got, ref):
        return np.linalg.norm(got.double().cpu().numpy() - ref) <= 1e-5 * np.linalg.norm(ref)
    for n in (room, room + 4 * Cin * Cout * K):
        guard = torch.full((n + 512,), 255, dtype=torch.uint8, device="cuda")
        assert near(nm.nm_conv1d_bwd_weight(xd, dyd, K, workspace=guard[:n], **kw), ref_dw)
        assert (guard[n:] == 255).all()
    guard = torch.full((both + 512,), 255, dtype=torch.uint8, device="cuda")
    dx, _, dw = nm.nm_conv1d_bwd(xd, dyd, wd, workspace=guard[:both], **kw)
    assert near(dw, ref_dw) and near(dx, ref_dx) and (guard[both:] == 255).all()


@pytest.mark.parametrize("dims", [(8, 205, 268, 393, 25, 1, 1, 12), (10, 250, 169, 668, 25, 1, 1, 12), (3, 97, 130, 500, 13, 1, 1, 6), (5, 33, 65, 711, 7, 2, 1, 3)],
                         ids=str)
def test_more_room_is_never_served_by_a_slower_kernel(dims):
    """Parts that are no multiple of 256 bytes: at every byte around the size of each number of parts."""
    import ctypes
    L, name = nm.lib(), ctypes.create_string_buffer(100)
    asked = nm.nm_conv1d_workspace_bytes(nm.NM_OP_BWD_WEIGHT, *dims, nm.NM_F32, 1)
    T_out = nm.nm_conv1d_out_len(dims[3], *dims[4:])
    g, part = -(-4 * dims[0] * dims[2] * T_out // 256) * 256, 4 * dims[1] * dims[2] * dims[4]
    assert part % 256 != 0
    fast = []
    for parts in range(1, 9):
        for n in range(g + parts * part - 300, g + parts * part + 301):
            assert L.nm_conv1d_kernel_name(nm.NM_OP_BWD_WEIGHT, *dims, nm.NM_F32, 1, 0, n, name, 100) == nm.NM_OK
            fast.append(name.value.startswith(b"f32_"))
            assert n < asked or fast[-1]
    assert fast == sorted(fast) and fast[-1] and not fast[0]
