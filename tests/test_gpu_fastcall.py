"""The per-layer calls through the native module and through ctypes are the same
call: equal bits for each function, and equal refusals."""
import pytest
import torch

from paper_1912_12675_amd import psw

pytestmark = pytest.mark.gpu


def _calls(rnd, res):
    """Every function once, the layers' outputs in a list."""
    n, c, k = 5, 12, 20
    x, w, b = rnd(n, c, 9, 9), rnd(k, c, 3, 3), rnd(k)
    y, dx, dw, db = rnd(n, k, 5, 5), rnd(n, c, 9, 9), rnd(k, c, 3, 3), rnd(k)
    psw.psw_conv_fwd(x, w, y, 2, 1, bias=b, relu=True)
    g = rnd(n, k, 5, 5)
    psw.psw_relu_mask(y, g)
    psw.psw_conv_bwd_data(x.shape, w, g, dx, 2, 1, accumulate=True)
    ws = torch.empty(max(1, psw.psw_conv_bwd_weight_ws_bytes(x.shape, w.shape, 2, 1)), dtype=torch.uint8, device="cuda")
    psw.psw_conv_bwd_weight(x, g, dw, 2, 1, dbias=db, ws=ws)
    gamma, beta, z, m, i = rnd(k), rnd(k), rnd(n, k, 5, 5), rnd(k), rnd(k)
    r = rnd(n, k, 5, 5) if res else None
    rm, rv = rnd(k), rnd(k)
    ws = torch.empty(max(1, psw.psw_bn_ws_bytes(y.shape)), dtype=torch.uint8, device="cuda")
    psw.psw_bn_relu_fwd(y, gamma, beta, z, m, i, res=r, relu=True, eps=1e-4, momentum=0.2, run_mean=rm, run_var=rv, ws=ws)
    dy, dg, dbt, dr = rnd(n, k, 5, 5), rnd(k), rnd(k), rnd(n, k, 5, 5) if res else None
    psw.psw_bn_relu_bwd(g, z, y, gamma, m, i, dy, dg, dbt, dres=dr, relu=True, res_accumulate=res, ws=ws)
    p, arg, dp = rnd(n, k, 2, 2), torch.zeros(n, k, 2, 2, dtype=torch.int32, device="cuda"), rnd(n, k, 5, 5)
    psw.psw_pool_fwd(psw.PSW_POOL_MAX, z, p, 2, 2, argmax=arg)
    psw.psw_pool_bwd(psw.PSW_POOL_MAX, z.shape, p, dp, 2, 2, argmax=arg, accumulate=True)
    f, fw, fb, o = rnd(n, 80), rnd(10, 80), rnd(10), rnd(n, 10)
    psw.psw_fc_fwd(f, fw, o, b=fb)
    lab = torch.arange(n, dtype=torch.int32, device="cuda")
    loss, dl = rnd(1), rnd(n, 10)
    psw.psw_softmax_xent(o, lab, loss, dl)
    dfx, dfw, dfb = rnd(n, 80), rnd(10, 80), rnd(10)
    ws = torch.empty(max(1, psw.psw_fc_bwd_ws_bytes(n, 80, 10)), dtype=torch.uint8, device="cuda")
    psw.psw_fc_bwd(f, fw, dl, dfw, dx=dfx, db=dfb, dx_accumulate=True, ws=ws)
    v, w2 = rnd(10, 80), rnd(10, 80)
    psw.psw_sgd_momentum_step(fw, w2, v, dfw, 0.05, 0.8, 0.01, nesterov=True)
    return [t for t in (y, g, dx, dw, db, z, m, i, rm, rv, dy, dg, dbt, dr, p, arg, dp, o, loss, dl, dfx, dfw, dfb, v, w2)
            if t is not None]


@pytest.mark.parametrize("res", [False, True])
def test_calls_equal(res, monkeypatch):
    def go():
        gen = torch.Generator(device="cuda").manual_seed(7)
        out = _calls(lambda *s: torch.randn(*s, generator=gen, device="cuda"), res)
        torch.cuda.synchronize()
        return out

    native = go()
    assert type(psw._fast).__name__ == "module"  # not already through ctypes
    monkeypatch.setattr(psw, "_fast", psw._CtypesOnly())
    for a, b in zip(native, go(), strict=True):
        assert torch.equal(a, b)


def test_current_stream():
    """Without a stream argument the call goes to the current one."""
    z, a = torch.zeros(1 << 20, device="cuda"), torch.ones(1 << 20, device="cuda")
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):  # a call on another stream would not be captured, but run
            psw.psw_relu_mask(z, a)
    torch.cuda.synchronize()
    assert bool((a == 1).all())
    g.replay()
    torch.cuda.synchronize()
    assert bool((a == 0).all())


def test_refusals():
    z = torch.ones(4, 4, device="cuda")
    with pytest.raises(ValueError, match="contiguous"):
        psw.psw_relu_mask(z, torch.ones(4, 4, device="cuda").t()[:, :2])
    with pytest.raises(TypeError):
        psw.psw_relu_mask(z, z.double())
    with pytest.raises(ValueError, match="device"):
        psw.psw_relu_mask(z, z.cpu())
    with pytest.raises(psw.PswError):
        x, w = torch.ones(1, 1, 4, 4, device="cuda"), torch.ones(1, 1, 3, 3, device="cuda")
        psw.psw_conv_fwd(x, w, torch.ones(1, 1, 4, 4, device="cuda"), stride=0, pad=1)
