"""The binding's two ways through: the native marshalling takes the usual call, everything else goes to the Python checks, and
both give the same results and refusals."""
import pytest
import torch

import paper_2302_06646_amd as lc

pytestmark = pytest.mark.gpu


def _layer(B=3, H=5, N=512, dt=torch.bfloat16):
    g = torch.Generator(device="cuda").manual_seed(7)
    r = lambda *s: torch.randn(*s, generator=g, device="cuda")
    u, dy, k, D = r(B, H, N).to(dt), r(B, H, N).to(dt), r(H, N) / N ** 0.5, r(H)
    ws = lc.new_workspace(B, H, N, lc.dtype_code(u), 1)
    return u, dy, k, D, ws


def _step(u, dy, k, D, ws, stream=None):
    y, du, dk, dD = torch.empty_like(u), torch.empty_like(u), torch.empty(k.shape, device="cuda"), torch.empty(len(D), device="cuda")
    ks = lc.new_kspec(k.shape[0], k.shape[1], lc.dtype_code(u))
    lc.longconv_kspec_compute(k, D, ks, lc.dtype_code(u), ws, stream=stream)
    lc.longconv_fwd(u, k, D, y, ws, kspec=ks, stream=stream)
    lc.longconv_bwd(dy, u, k, D, du, dk, dD, ws, kspec=ks, stream=stream)
    torch.cuda.synchronize()
    return y, du, dk, dD


class _Sub(torch.Tensor):
    pass


def test_every_way_through_gives_the_same_bits():
    u, dy, k, D, ws = _layer()
    want = _step(u, dy, k, D, ws)
    n = lc._fast()
    assert n.kspec_compute(k, D, lc.new_kspec(5, 512, lc.BF16), lc.BF16, ws, None) == 0           # taken natively
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    ways = [
        _step(u, dy, torch.nn.Parameter(k), torch.nn.Parameter(D), ws),                           # parameters
        _step(u, dy, k, D, ws, stream=s),                                                         # a stream object
        _step(u.as_subclass(_Sub), dy, k, D, ws),                                                 # a subclass: the Python way
    ]
    assert n.fwd(u.as_subclass(_Sub), k, D, torch.empty_like(u), ws, None, None) is None
    with torch.cuda.stream(s):
        ways.append(_step(u, dy, k, D, ws))
    for got in ways:
        for a, b in zip(got, want):
            assert torch.equal(a.as_subclass(torch.Tensor), b)


def test_what_was_refused_stays_refused():
    u, dy, k, D, ws = _layer()
    y = torch.empty_like(u)
    bad = [
        (u, k, D, torch.empty(3, 5, 256, dtype=u.dtype, device="cuda"), ws),      # shape of the output
        (u, k.half(), D, y, ws),                                                  # dtype of the kernel
        (u.transpose(0, 1).contiguous().transpose(0, 1), k, D, y, ws),            # strides
        (u.cpu(), k, D, y, ws),                                                   # device
        (u, k, D, None, ws),                                                      # no output
        (u, k, D, y, ws[:64]),                                                    # workspace too small
        (u, k, D, y.view(-1)[4:4 + 3 * 5 * 256].view(3, 5, 256), ws),             # shape again, off alignment
    ]
    for args in bad:
        with pytest.raises(lc.LongconvError):
            lc.longconv_fwd(*args)
    with pytest.raises(AttributeError):
        lc.longconv_fwd(u, k, D, y, None)
    with pytest.raises(ValueError):
        lc.longconv_fwd(u[0], k, D, y, ws)
    with pytest.raises(KeyError):
        lc.longconv_fwd(u.double(), k, D, y, ws)
    with torch.no_grad():
        batched = torch.func.vmap(lambda v: lc.longconv_fwd(v, k, D, y, ws) or v)
        with pytest.raises(Exception):
            batched(torch.stack([u, u]))                                          # no storage to point at
    torch.cuda.synchronize()
