"""Where initial values come from. daic_problem_set_init_device takes what a copy takes: aligned arrays of the
state's device (read by a kernel), and arrays at odd addresses, in pinned and
in ordinary host memory (copied); daic_problem_set_init takes host arrays by a
plain copy from 16 KiB to 12 MiB and through pinned chunks otherwise."""
import ctypes

import numpy as np
import pytest

from test_gpu_transfer import empty_graph, roundtrip, weighted_graph

pytestmark = pytest.mark.gpu

daic = pytest.importorskip("paper_1710_05785_amd.daic")
torch = pytest.importorskip("torch")


def place(x, where):
    """(address of a copy of x, what keeps it alive)"""
    raw = torch.from_numpy(x.view(np.uint8).copy())
    if where == "pinned":
        raw = raw.pin_memory()
    elif where != "host":
        at = {"device": 0, "odd": 3}[where]
        buf = torch.zeros(raw.numel() + 16, dtype=torch.uint8, device="cuda")
        buf[at:at + raw.numel()] = raw.cuda()
        return buf.data_ptr() + at, buf
    return raw.data_ptr(), raw


@pytest.mark.parametrize("where", [("device", "device"), ("device", "odd"), ("odd", "device"), ("pinned", "device"),
                                   ("device", "host"), ("host", "host")])
@pytest.mark.parametrize("state", ["f64", "f32_kahan", "u32"])
def test_arrays_of_any_memory(state, where):
    n = 70001
    rng = np.random.default_rng(n)
    if state == "u32":
        p = daic.Problem(weighted_graph(n), daic.MIN, daic.G_EDGE_ADD, state=state)
        v, dv = (rng.integers(0, 1 << 32, n, dtype=np.uint32) for _ in range(2))
    else:
        p = daic.Problem(empty_graph(n), daic.SUM, daic.G_SRC_SCALE, alpha=0.5, state=state)
        v, dv = (rng.standard_normal(n).astype(np.float64 if state == "f64" else np.float32) for _ in range(2))
        p.set_init(v.astype(np.float64) + 1e-9, dv.astype(np.float64))  # (a compensation that the call clears)
    (a, keep_a), (b, keep_b) = place(v, where[0]), place(dv, where[1])
    torch.cuda.synchronize()
    call = daic.lib().daic_problem_set_init_device
    daic.check(call(p._h, ctypes.c_void_p(a), ctypes.c_void_p(b), None), "set_init_device")
    got_v, got_dv = p.get(with_dv=True)
    np.testing.assert_array_equal(got_v, v.astype(got_v.dtype))
    np.testing.assert_array_equal(got_dv, dv.astype(got_dv.dtype))
    del keep_a, keep_b


@pytest.mark.parametrize("state", ["f64", "u32"])
@pytest.mark.parametrize("more", [-1, 0, 1])
def test_host_arrays_around_the_limits_of_plain_copies(state, more):
    for limit in (16 << 10, 12 << 20):
        assert roundtrip(limit // (8 if state == "f64" else 4) + more, state)
