"""GPU parity of rtc_cfr_loss_adjoint_cir where its route changes with a
link's delays: the number of node blocks (16 taps each), the widest span the
nodes take (116 taps), wider spans and delays beyond the window (paths
contracted directly), links of one path and of none; against the FP64 oracle's
reverse-mode gradient.  Tolerances as for the fused pass with H* targets: loss
1e-5; dL/da 3e-5 normwise and 1e-4 per link; dL/dg 3e-5."""
import numpy as np
import pytest
import torch

from oracle import channel as och

pytestmark = pytest.mark.gpu
c128 = torch.complex128

# subcarriers, elements, per link: paths, first delay and span in taps
CASES = {
    "blocks_n1024_m32": (1024, 32, [(40, 3.25, 3.0), (33, 7.0, 3.999), (70, 20.5, 4.0),
                                    (64, 100.0, 19.5), (65, 0.01, 36.5), (200, 11.0, 52.5),
                                    (31, 500.0, 68.5)]),
    "edge_of_nodes_n512_m7": (512, 7, [(50, 5.0, 115.999), (50, 5.0, 116.001), (90, 30.0, 116.0),
                                       (40, 0.5, 117.0), (70, 5.25, 99.0)]),
    "direct_n256_m32": (256, 32, [(37, 0.0, 200.0), (100, 10.0, 255.0), (64, 3.0, 120.0),
                                  (33, 200.0, 700.0)]),
    "direct_n1024_m3": (1024, 3, [(96, 0.0, 1023.0), (20, 900.0, 300.0)]),
    "beyond_the_window_n256_m4": (256, 4, [(40, 250.0, 20.0), (40, 1000.5, 30.0),
                                           (12, 5000.0, 8.0)]),
    "few_paths_n512_m32": (512, 32, [(1, 12.0, 0.0), (0, 0.0, 0.0), (2, 30.5, 0.0),
                                     (1, 17.25, 0.0), (0, 0.0, 0.0), (3, 2.0, 60.0)]),
    "on_the_taps_n1024_m1": (1024, 1, [(16, 8.0, -1.0), (16, 8.5, -1.0)]),
}


@pytest.fixture(scope="module")
def rl(gpu_lib):
    from paper_2311_18558_amd import lib
    return lib


def _inputs(N, M, links, seed=5):
    rng = np.random.default_rng(seed)
    taps = [x0 + (np.arange(n, dtype=float) if span < 0 else
                  np.concatenate([[0.0, span][:n], rng.uniform(0, 1, max(0, n - 2)) * span]))
            for n, x0, span in links]
    off = np.concatenate([[0], np.cumsum([len(t) for t in taps])]).astype(np.int64)
    x = np.concatenate(taps)
    a = (rng.normal(size=len(x)) + 1j * rng.normal(size=len(x))) * 1e-4 / (1 + 0.05 * x)
    g = rng.uniform(0.8, 1.2, M) * np.exp(1j * rng.uniform(-0.7, 0.7, M))
    return off, x, a.astype(np.complex64), rng.uniform(-np.pi, np.pi, len(x)).astype(np.float32), \
        g.astype(np.complex64)


@pytest.mark.parametrize("case", list(CASES))
def test_delay_routes_against_oracle(rl, case):
    from types import SimpleNamespace
    N, M, links = CASES[case]
    off, x, a, psi, g = _inputs(N, M, links)
    L, P, bw, fc = len(links), len(x), 50e6, 3.5e9
    tau = x / bw
    f = och.subcarrier_freqs(fc, bw, N)
    a64 = torch.tensor(a).to(c128).requires_grad_(True)
    g64 = torch.tensor(g).to(c128).requires_grad_(True)
    psi64 = torch.tensor(psi).double()
    Ht = och.cfr(off, tau, a64.detach() * 1.1 * np.exp(0.2j), psi64, g64.detach(), f)
    Ht = Ht.to(torch.complex64)
    tot, coh, inc = och.cfr_loss(och.cfr(off, tau, a64, psi64, g64, f), Ht.to(c128))
    da_ref, dg_ref = torch.autograd.grad(tot, (a64, g64))

    D = 1
    z = np.zeros((3, D * P), np.float32)
    dp = rl.DevicePaths(SimpleNamespace(
        n_links=L, n_paths=P, max_depth=D, link_off=off, tx_pos=np.zeros((L, 3)),
        rx_pos=np.ones((L, 3)), depth=np.zeros(P, np.uint8), pts=z, nrm=z,
        mat=np.zeros(D * P, np.uint16), kind=np.zeros(D * P, np.uint8),
        dA=np.zeros(D * P, np.float32), tau=tau))
    rc = rl.make_radio(fc, bw / N, N, M)
    stats = torch.empty(2, dtype=torch.float64, device="cuda")
    X = torch.empty((L, M, N), dtype=torch.complex64, device="cuda")
    ws = rl.workspace(rl.RTC_OP_CFR_TARGET_STATS, rc, L, P)
    rl.cfr_target_cir(rc, L, Ht.cuda(), stats, X, ws)
    loss = torch.full((3,), float("nan"), dtype=torch.float64, device="cuda")
    da = torch.full((P,), float("nan"), dtype=torch.complex64, device="cuda")
    dg = torch.full((M,), float("nan"), dtype=torch.complex64, device="cuda")
    rl.cfr_loss_adjoint_cir(rc, dp, torch.tensor(a).cuda(), torch.tensor(psi).cuda(),
                            torch.tensor(g).cuda(), X, stats, 1.0, 1.0, loss, da, dg,
                            rl.workspace(rl.RTC_OP_CFR_LOSS_ADJOINT, rc, L, P))
    torch.cuda.synchronize()
    for got, ref in zip(loss.tolist(), (tot.item(), coh.item(), inc.item())):
        assert abs(got - ref) <= 1e-5 * abs(ref), (got, ref)
    rel = lambda u, v: (torch.linalg.norm(u - v) / torch.linalg.norm(v)).item()  # noqa: E731
    da, dg = da.cpu().to(c128), dg.cpu().to(c128)
    worst = max(rel(da[off[l]:off[l + 1]], da_ref[off[l]:off[l + 1]])
                for l in range(L) if off[l + 1] > off[l])
    print(f"[gpu-step] {case}: dL/da {rel(da, da_ref):.2e} (per link {worst:.2e}), "
          f"dL/dg {rel(dg, dg_ref):.2e}", flush=True)
    assert rel(da, da_ref) <= 3e-5 and worst <= 1e-4 and rel(dg, dg_ref) <= 3e-5


def test_delay_that_is_not_finite(rl):
    """A link with a NaN delay gives NaN gradients for its paths and a NaN
    loss; the other links' gradients are untouched."""
    from types import SimpleNamespace
    N, M, links = 256, 4, [(20, 5.0, 10.0), (20, 5.0, 10.0)]
    off, x, a, psi, g = _inputs(N, M, links)
    out = []
    for bad in (False, True):
        tau = x / 50e6
        if bad:
            tau[3] = np.nan
        z = np.zeros((3, len(x)), np.float32)
        dp = rl.DevicePaths(SimpleNamespace(
            n_links=2, n_paths=len(x), max_depth=1, link_off=off, tx_pos=np.zeros((2, 3)),
            rx_pos=np.ones((2, 3)), depth=np.zeros(len(x), np.uint8), pts=z, nrm=z,
            mat=np.zeros(len(x), np.uint16), kind=np.zeros(len(x), np.uint8),
            dA=np.zeros(len(x), np.float32), tau=tau))
        rc = rl.make_radio(3.5e9, 50e6 / N, N, M)
        X = torch.ones((2, M, N), dtype=torch.complex64, device="cuda") * 1e-3
        stats = torch.ones(2, dtype=torch.float64, device="cuda")
        loss = torch.empty(3, dtype=torch.float64, device="cuda")
        da = torch.empty(len(x), dtype=torch.complex64, device="cuda")
        rl.cfr_loss_adjoint_cir(rc, dp, torch.tensor(a).cuda(), torch.tensor(psi).cuda(),
                                torch.tensor(g).cuda(), X, stats, 1.0, 1.0, loss, da, None,
                                rl.workspace(rl.RTC_OP_CFR_LOSS_ADJOINT, rc, 2, len(x)))
        torch.cuda.synchronize()
        out.append((loss.cpu(), da.cpu()))
    (l0, d0), (l1, d1) = out
    assert torch.isfinite(l0).all() and torch.isnan(l1[0])
    assert torch.isnan(torch.view_as_real(d1[:20])).any()
    assert torch.equal(d0[20:], d1[20:])
