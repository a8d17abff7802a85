"""The corrector's fused kernels where their tiles can go wrong: images of one
tile (whose halo wraps onto itself), of odd and few channels, several images,
volumes that start off any 16-byte boundary, and in place, against the network
in float64 with the operands rounded to bfloat16 as the kernels round them.

Every product is exact in FP32 and sums of 288 terms carry at most 288 * 6e-8
relative to the sum of magnitudes; a hidden activation that this moves across a
rounding boundary of bfloat16 changes by 2^-8 of itself, which few do.  The
residual then agrees to about one bfloat16 rounding, 2^-8 relative to its rms,
and the gradients, sums of products of such values, to the same 2^-8."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

C = 32
TOL = 2.0 ** -8


def _bf(x):
    return x.float().to(torch.bfloat16).double()


def _params(N, seed):
    rng = np.random.default_rng(seed)
    W = (rng.standard_normal((3, C, C, 9)) / np.sqrt(9 * C / 2)).astype(np.float32)
    b = (0.1 * rng.standard_normal((3, C))).astype(np.float32)
    W[0, :, N:] = 0
    W[2, N:] = 0
    b[2, N:] = 0
    return W, b


def _conv(a, W):
    """a [B][C][M][M], W [o][c][9] float64: the circular cross-correlation."""
    out = 0
    for tap in range(9):
        s = torch.roll(a, (1 - tap // 3, 1 - tap % 3), (2, 3))
        out = out + torch.matmul(W[:, :, tap], s.reshape(a.shape[0], C, -1)).reshape(a.shape)
    return out


def _net(psi, W, b):
    """Residual and the packed activations, all float64 on the CPU."""
    B, N, M, _ = psi.shape
    scale = psi.double().square().mean((1, 2, 3)).sqrt().float().double()
    Wr = [_bf(torch.from_numpy(W[i])) for i in range(3)]
    br = [torch.from_numpy(b[i]).double().view(1, C, 1, 1) for i in range(3)]
    a0 = torch.zeros(B, C, M, M, dtype=torch.float64)
    a0[:, :N] = _bf(psi.double() / scale.view(-1, 1, 1, 1))
    a1 = _bf(torch.relu(_conv(a0, Wr[0]) + br[0]))
    a2 = _bf(torch.relu(_conv(a1, Wr[1]) + br[1]))
    r = (_conv(a2, Wr[2]) + br[2])[:, :N]
    return scale, Wr, (a0, a1, a2), r


def _offset(x, off):
    """The same values in a contiguous tensor `off` floats into its storage."""
    buf = torch.empty(x.numel() + off, dtype=x.dtype, device="cuda")
    v = buf[off:].view(x.shape)
    v.copy_(x)
    return v


CASES = [(16, 1, 1), (16, 32, 3), (32, 17, 1), (48, 5, 2), (80, 31, 1)]


@pytest.mark.parametrize("M,N,B", CASES)
def test_network_on_small_tiles(M, N, B):
    from paper_1304_2062_amd import se2n
    print(f"cnn tiles {M} {N} {B}", flush=True)
    W, b = _params(N, M + N)
    net = se2n.Corrector(N, seed=1)
    net.set_params(np.concatenate([np.concatenate([W[i].ravel(), b[i]]) for i in range(3)]))
    g = torch.Generator().manual_seed(M * N)
    psi = torch.rand(B, N, M, M, generator=g)
    scale, _, _, r = _net(psi, W, b)
    net.workspace(M, B, False).fill_(255)  # NaN bytes: nothing is read before it is written
    for off in (0, 1):
        x = _offset(psi, off)
        got = net.forward(x, _offset(torch.zeros_like(psi), off))
        res = (got.cpu().double() - psi.double()) / scale.view(-1, 1, 1, 1)
        assert float((res - r).norm() / r.norm()) < TOL
        assert torch.equal(net.forward(x, x), got)  # in place: the same arithmetic


@pytest.mark.parametrize("M,N,B", CASES)
def test_gradients_on_small_tiles(M, N, B):
    from paper_1304_2062_amd import se2n
    print(f"cnn gradients {M} {N} {B}", flush=True)
    W, b = _params(N, M + N)
    net = se2n.Corrector(N, seed=1)
    net.set_params(np.concatenate([np.concatenate([W[i].ravel(), b[i]]) for i in range(3)]))
    g = torch.Generator().manual_seed(M * N + 1)
    psi = torch.rand(B, N, M, M, generator=g)
    fine = torch.rand(B, N, M, M, generator=g)
    scale, Wr, acts, r = _net(psi, W, b)
    sc = scale.view(-1, 1, 1, 1)
    d = torch.zeros(B, C, M, M, dtype=torch.float64)
    d[:, :N] = (psi.double() + sc * r - fine.double()) / sc
    loss = float(d.square().sum() / psi.numel())
    want = []
    gr = _bf(2.0 / psi.numel() * d)
    for layer in (2, 1, 0):
        a = acts[layer]
        dW = torch.stack([torch.matmul(gr.permute(1, 0, 2, 3).reshape(C, -1),
                                       torch.roll(a, (1 - t // 3, 1 - t % 3), (2, 3)).permute(1, 0, 2, 3)
                                       .reshape(C, -1).T) for t in range(9)], 2)
        want.insert(0, torch.cat([dW.reshape(-1), gr.sum((0, 2, 3))]))
        if layer:
            back = Wr[layer].flip(2).permute(1, 0, 2)
            gr = _bf(torch.where(a > 0, _conv(gr, back), torch.zeros(())))
    net.workspace(M, B, True).fill_(255)
    grads, got_loss = net.gradients(_offset(psi, 1), _offset(fine, 1))
    assert abs(float(got_loss) - loss) < TOL * loss
    n = C * C * 9 + C
    for layer in range(3):
        got = grads.cpu().double()[layer * n:(layer + 1) * n]
        assert float((got - want[layer]).norm() / want[layer].norm()) < TOL
