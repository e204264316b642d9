"""The binding's tensor checks: its combined test of the usual case accepts nothing
the full checks refuse, and tensors it does not take (subclasses, other strides of
size-1 dimensions) still pass through the full checks."""

import copy

import pytest
import torch

from paper_2609_33503_amd import relaxkv

pytestmark = pytest.mark.gpu


def test_binding_checks(gpu_lib):
    L, Qn, H, Hkv, T, d = 1, 3, 4, 2, 40, 64
    bf = dict(dtype=torch.bfloat16, device="cuda")
    q, k = torch.randn(L, Qn, H, d, **bf), torch.randn(L, Hkv, T, d, **bf)
    kq, out = torch.randn(Qn, Hkv, d, **bf), torch.empty(Qn, H, d, **bf)
    lse = torch.empty(Qn, H, device="cuda")
    req = relaxkv.Request(q, k, k.clone(), 0.2)
    ws = req.alloc_query_workspace()
    good = dict(k_cache=k, v_cache=k, k_q=kq, v_q=kq, out=out, lse_out=lse, ws=ws)
    req.query_attn(0, **good)
    ref = out.clone()
    # a subclass, and a cache whose size-1 layer dimension has another stride
    p = torch.nn.Parameter(kq, requires_grad=False)
    req.query_attn(0, **{**good, "k_q": p, "k_cache": k.as_strided(k.shape, (7,) + k.stride()[1:])})
    assert torch.equal(out, ref)
    req.query_attn(0, **good, stream=torch.cuda.current_stream())
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):                      # the current stream is the one used
        out.zero_()
        req.query_attn(0, **good)
        got = out.clone()
    torch.cuda.current_stream().wait_stream(side)
    assert torch.equal(got, ref)
    wide = torch.empty(Qn, H, 2 * d, **bf)
    bad = [dict(k_q=kq.float()), dict(k_q=kq[:2]), dict(k_q=kq.cpu()), dict(k_q=None),
           dict(out=wide[:, :, :d]), dict(lse_out=lse.double()), dict(lse_out=lse.t()),
           dict(k_cache=k[:, :, :-1]), dict(v_cache=k.cpu()), dict(v_cache=k.float()),
           dict(v_cache=k.transpose(1, 2).contiguous().transpose(1, 2)),
           dict(ws=ws.cpu()), dict(ws=ws[::2])]
    for b in bad:
        with pytest.raises(ValueError):
            req.query_attn(0, **{**good, **b})
    sets = req.alloc_sets()
    a = torch.rand(L, T, device="cuda")
    for b in (a.cpu(), a.double(), a[:, :-1], a.t(), [0.0]):
        with pytest.raises(ValueError):
            req.select(b, sets)
    req.select(a, sets)
    req.build_sets(sets)
    n = int(sets.counts[1])
    r = [torch.randn(n, h, d, **bf) for h in (H, Hkv, Hkv, H)]
    req.sparse_attn(sets, 0, *r)
    for i in range(4):
        for x in (r[i][:-1], r[i].cpu(), r[i].float(), None):
            with pytest.raises(ValueError):
                req.sparse_attn(sets, 0, *(x if j == i else t for j, t in enumerate(r)))
    with pytest.raises(ValueError):
        req.update_cache(sets, 0, r[1], r[2][:-1], k, k)
    torch.cuda.synchronize()


def test_calls_use_the_request_s_descriptor(gpu_lib):
    """A request whose descriptor is replaced (a copy with another softmax scale)
    runs with the new one, and the request it was copied from with its own."""
    L, Qn, H, Hkv, T, d = 2, 3, 4, 2, 70, 64
    bf = dict(dtype=torch.bfloat16, device="cuda")
    q, k = torch.randn(L, Qn, H, d, **bf), torch.randn(L, Hkv, T, d, **bf)
    kq = torch.randn(Qn, Hkv, d, **bf)

    def results(req):
        a, out = torch.empty(L, T, device="cuda"), torch.empty(Qn, H, d, **bf)
        req.score(req.alloc_workspace(), a)
        req.query_attn(1, k, k, kq, kq, out, ws=req.alloc_query_workspace())
        return a, out
    req = relaxkv.Request(q, k, k, 0.2)
    other = copy.copy(req)
    other.p = relaxkv.Problem.from_buffer_copy(req.p)
    other.p.softmax_scale = 0.5
    want = [results(relaxkv.Request(q, k, k, 0.2, softmax_scale=s)) for s in (0.0, 0.5)]
    for got, ref in zip((results(req), results(other)), want):
        assert torch.equal(got[0], ref[0]) and torch.equal(got[1], ref[1])
    assert not torch.equal(want[0][1], want[1][1])
