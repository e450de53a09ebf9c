"""The one call behind the binding's products: what it refuses, and that it is the product it names."""
import numpy as np
import pytest

import paper_2504_08860_amd as H


def test_no_handle_is_an_invalid_argument():
    for kind in (-1, 0, 1, 2, 3):
        assert H.lib().hbp_spmv_sized(None, kind, None, 0, None, 0, None) == -1
    assert "long" in H.hbp_status_string(H.HBP_ERR_WRONG_LENGTH)


@pytest.mark.parametrize("gone", ["_cuda_getCurrentRawStream", "_cuda_getDevice"])
def test_a_torch_without_its_private_calls(monkeypatch, gone):
    """The current stream is asked for in public where either is missing."""
    import types

    import torch
    H.lib()
    for name in ("_lib", "_torch", "_raw_stream", "_device"):
        monkeypatch.setattr(H, name, getattr(H, name))      # (as they were, afterwards)
    for name in ("_cuda_getCurrentRawStream", "_cuda_getDevice"):
        monkeypatch.setattr(torch._C, name, lambda *_: 5, raising=False)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=77))
    H._lib = None
    H.lib()
    assert H._stream_ptr(None) == 5
    monkeypatch.delattr(torch._C, gone)
    H._lib = None
    H.lib()
    assert H._stream_ptr(None) == 77


@pytest.mark.gpu
@pytest.mark.parametrize("kind", [0, 1, 2])
def test_products_by_kind(kind):
    import torch
    from workloads import random_csr, widen_to_f64
    m = random_csr(300, 200, 0.05, 3)
    m = widen_to_f64(m) if kind == 1 else m
    call, build = [(H.hbp_spmv, H.hbp_build), (H.hbp_spmv_f64, H.hbp_build_f64), (H.hbp_spmv_static_scratch, H.hbp_build)][kind]
    t = lambda a: torch.from_numpy(a).cuda()  # noqa: E731
    h = build(t(m.ptr), t(m.col), t(m.val), m.n_rows, m.n_cols)
    try:
        x, y = t(m.x), torch.full((m.n_rows,), float("nan"), dtype=t(m.x).dtype, device="cuda")
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        for stream in (None, side, side.cuda_stream):
            y.fill_(float("nan"))
            side.wait_stream(torch.cuda.current_stream())
            call(h, x, y, stream)
            torch.cuda.synchronize()
            want = np.zeros(m.n_rows)
            np.add.at(want, np.repeat(np.arange(m.n_rows), np.diff(m.ptr)), m.val.astype(np.float64) * m.x.astype(np.float64)[m.col])
            assert np.allclose(y.cpu().numpy(), want, rtol=1e-5, atol=1e-5)
        with torch.cuda.stream(side):  # torch's current stream is where a call without one goes
            y.fill_(float("nan"))
            call(h, x, y)
            assert not torch.isnan(y).any()
        torch.cuda.synchronize()
        for bad_x, bad_y in ((x[:-1], y), (x, y[:-1]), (torch.cat([x, x]), y)):
            with pytest.raises(AssertionError):
                call(h, bad_x, bad_y)
        with pytest.raises(AssertionError):
            call(h, x.to(torch.float16), y)
        with pytest.raises(AssertionError):
            call(h, x.cpu(), y)
        with pytest.raises(H.HbpError):
            call(None, x, y)
        other = H.hbp_spmv if kind == 1 else H.hbp_spmv_f64  # the other value type's handle
        with pytest.raises((AssertionError, H.HbpError)):
            other(h, x, y)
        with pytest.raises(H.HbpError):
            z = torch.zeros(m.n_cols, dtype=torch.float32 if kind == 1 else torch.float64, device="cuda")
            other(h, z, torch.zeros(m.n_rows, dtype=z.dtype, device="cuda"))
    finally:
        H.hbp_free(h)
