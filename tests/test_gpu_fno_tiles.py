"""The network's layer kernels at the edges of their tiles: grids of 1 to 64 row
blocks (a column tile of 32 is cut at N = 16, 48, 144), one to 32 modes (one or two 16-blocks of
modes), one to 32 channels (odd counts, the second 16-block of channels), rows of the outputs not
a multiple of 4, and inputs and targets at addresses that are not 16-byte aligned."""
import numpy as np
import pytest

from oracle import fno_oracle as F

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

CASES = [F.Config(N=16, m=1, w=1, L=0, p=1), F.Config(N=16, m=16, w=17, L=1, p=3),
         F.Config(N=32, m=32, w=16, L=1, p=16), F.Config(N=48, m=17, w=31, L=1, p=5),
         F.Config(N=48, m=5, w=3, L=2, p=17), F.Config(N=144, m=31, w=9, L=1, p=8),
         F.Config(N=144, m=16, w=32, L=1, p=32), F.Config(N=272, m=20, w=5, L=1, p=31),
         F.Config(N=1024, m=32, w=1, L=0, p=1)]


def _at(a, shift):
    """a on the device, float32, `shift` elements past a 256-byte boundary."""
    buf = torch.zeros(a.size + shift, dtype=torch.float32, device="cuda")
    buf[shift:] = torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float32).reshape(-1).cuda()
    return buf[shift:].view(a.shape)


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("cfg", CASES, ids=lambda c: f"N{c.N}m{c.m}w{c.w}p{c.p}")
def test_layers_at_tile_edges(cfg, shift):
    """Forward within 2e-5 of the largest output; the gradient within 1e-3 of its group's largest
    entry, plus what the float32 rounding of Y (1e-6) becomes through (Y^T Y)^-1."""
    from paper_2306_10379_amd import fno
    B = 2
    g = np.random.default_rng(cfg.N + cfg.m + cfg.w)
    flat = (0.3 * g.standard_normal(F.param_count(cfg))).astype(np.float32)
    V = (-20.0 * g.random((B, cfg.N * cfg.N))).astype(np.float32)
    X = np.stack([np.linalg.qr(g.standard_normal((cfg.N * cfg.N, cfg.p)))[0] for _ in range(B)]).astype(np.float32)
    net = fno.Net(N=cfg.N, modes=cfg.m, width=cfg.w, layers=cfg.L, p=cfg.p, max_batch=B)
    net.set_params(_at(flat, 0))
    f64 = [a.astype(np.float64) for a in (flat, V, X)]
    Yref = np.asarray(F.predict(f64[0], f64[1], cfg)).reshape(B, -1, cfg.p)
    Y = net.forward(_at(V, shift)).double().cpu().numpy().reshape(Yref.shape)
    print(f"fno {cfg} shift {shift}: forward {np.max(np.abs(Y - Yref)) / np.max(np.abs(Yref)):.1e}", flush=True)
    assert np.max(np.abs(Y - Yref)) <= 2e-5 * np.max(np.abs(Yref))
    loss, grad = net.loss_grad(_at(V, shift), _at(X, shift))
    _, gref, per = F.loss_and_grad(*f64, cfg)
    cond = max(np.linalg.cond(y.T @ y) for y in Yref)
    assert np.allclose(loss, per, rtol=1e-4, atol=1e-5)
    got, off = grad.double().cpu().numpy(), 0
    for name, shape in F.param_shapes(cfg):
        size = int(np.prod(shape))
        ref = gref[off:off + size]
        assert np.max(np.abs(got[off:off + size] - ref)) <= (1e-3 + 1e-6 * cond) * np.max(np.abs(ref)) + 1e-7, name
        off += size
    net.close()
