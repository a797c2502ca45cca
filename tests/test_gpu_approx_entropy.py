"""Large bf16 tensors are ranked from approximate entropies, and the tiles near the threshold from exact ones: the stream must be the one
that the multi-launch selection writes, which ranks all tiles by their exact entropies."""
import math

import numpy as np
import pytest
import torch

import paper_2506_01352_amd as tahq

pytestmark = pytest.mark.gpu

ELEMENTS = 1 << 25                                       # from here on entropies are approximate


def _both_ways(cfg, x):
    codec = tahq.Codec(cfg, device="cuda")
    codec.workspace.fill_(0xFF)
    codec.packed.fill_(0xFF)
    tahq.tahq_encode(cfg, x, codec.packed, codec.workspace)
    fused = codec.packed.clone()
    codec.workspace.fill_(0xFF)
    tahq.tahq_encode_phases(cfg, x, codec.packed, codec.workspace, tahq.PHASE_ALL | tahq.SELECT_MULTI_LAUNCH)
    torch.cuda.synchronize()
    assert torch.equal(fused, codec.packed), "the two selections differ"
    return fused


def _approximate(cfg, x):
    """The entropies that the selection starts from: the scratch behind its counters, histograms and candidate lists."""
    codec = tahq.Codec(cfg, device="cuda")
    for phase in (tahq.PHASE_PROLOGUE, tahq.PHASE_ENTROPY):
        tahq.tahq_encode_phases(cfg, x, codec.packed, codec.workspace, phase)
    tiles = cfg.batch * cfg.seq * cfg.hidden // cfg.tile
    units = 1 if cfg.scope else cfg.batch

    def pad256(v):
        return (v + 255) // 256 * 256
    at = pad256(units * (512 + 32 + 4096 + 8192 + 16))
    at = pad256(at + units * 2 * min(-(-tiles // units // 8192), 64) * 2048 * 4)
    at = pad256(at + units * 16384 * 8)
    torch.cuda.synchronize()
    return codec.workspace[at:at + 4 * tiles].view(torch.float32).clone()


def _exact(cfg, x):
    H = torch.empty(cfg.batch * cfg.seq * cfg.hidden // cfg.tile, device="cuda")
    tahq.tahq_tile_entropy(cfg, x, H)
    return H


SLACK = 7e-5                                             # derived beside the kernel's constant of that value


def _normal(shape, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return torch.randn(shape, device="cuda", generator=g), g


@pytest.mark.parametrize("G", (8, 16, 32, 64, 128))
@pytest.mark.parametrize("shape,scope", (((2, 2048, 8192), 0), ((1, 4096, 8192), 1), ((3, 2731, 4128), 0)))
def test_ordinary_values(G, shape, scope):
    # whole tensors and samples as ranking units; the last shape's units are no multiple of 64 tiles
    B, S, C = shape
    C = C // G * G
    S = max(S, -(-ELEMENTS // (B * C)))
    x, g = _normal((B, S, C), G)
    x = (x * torch.exp(0.5 * torch.randn(B, S, 1, device="cuda", generator=g))).to(torch.bfloat16)
    for budget in (3.2, 3.77):
        print(f"[case] ordinary [{B},{S},{C}] G={G} scope={scope} budget {budget}", flush=True)
        _both_ways(tahq.make_config(B, S, C, G, tahq.BF16, budget, scope=scope), x)


@pytest.mark.parametrize("G", (8, 64, 128))
@pytest.mark.parametrize("share", (0.028, 0.3))
def test_thresholds_in_and_beside_a_crowd_of_nearly_alike_tiles(G, share):
    # tiles that are one tile's elements in another order, with other signs and another power of two: their entropies differ in the last
    # bits only, far less than the approximation is off.  Thresholds from two bins below them to two above, where the bins
    # beside the threshold's may or may not hold more candidates than are listed.
    S, C = ELEMENTS // 8192, 8192
    n = S * C // G
    x, g = _normal((n, G), 7)
    crowd = torch.randperm(n, device="cuda", generator=g)[:int(share * n)]
    one = x[0].sort().values
    order = torch.rand(crowd.numel(), G, device="cuda", generator=g).argsort(1)
    sign = torch.randint(0, 2, (crowd.numel(), G), device="cuda", generator=g) * 2.0 - 1.0
    power = torch.exp2(torch.randint(-6, 7, (crowd.numel(), 1), device="cuda", generator=g).float())
    x[crowd] = one[order] * sign * power
    x = x.to(torch.bfloat16).reshape(1, S, C)
    H = torch.empty(n, device="cuda")
    tahq.tahq_tile_entropy(tahq.make_config(1, S, C, G, tahq.BF16, 3.5), x, H)
    at, width = H[crowd].median().item(), math.log(G) / 2048
    for bins in (-2.1, -1.02, -0.98, -0.5, -0.02, 0.0, 0.02, 0.5, 0.98, 1.02, 2.1):
        k = int((H > at + bins * width).sum()) + 3
        print(f"[case] G={G} {share} alike, threshold {bins} bins from them", flush=True)
        _both_ways(tahq.make_config(1, S, C, G, tahq.BF16, float(np.float32(3.0 + k / n))), x)


@pytest.mark.parametrize("G", (16, 64))
def test_values_outside_the_approximation(G):
    # zero tiles, tokens so small or large that products would leave fp32, elements below the normal numbers, tokens of five
    # elements, and numbers that are none
    B, S, C = 1, ELEMENTS // 8192, 8192
    x, g = _normal((B, S, C), 3)
    x[:, ::7] = 0.0
    x[:, 1::11] *= 1e-12
    x[:, 2::13] *= 1e30
    x[:, 3::17] *= 1e-39
    x[:, 4::19, 5:] = 0.0
    x[:, 5::23, ::2] *= 1e-38
    x = x.to(torch.bfloat16)
    for budget in (3.1, 3.6, 3.95):
        print(f"[case] outside, G={G} budget {budget}", flush=True)
        _both_ways(tahq.make_config(B, S, C, G, tahq.BF16, budget), x)
    x[0, 9, 3], x[0, 100, 70], x[0, 101, 130] = float("nan"), float("inf"), float("-inf")
    x[0, 200:240, :G] = float("nan")
    print(f"[case] outside, not finite, G={G}", flush=True)
    _both_ways(tahq.make_config(B, S, C, G, tahq.BF16, 3.6), x)


@pytest.mark.parametrize("eps_l1,eps_log", ((1e-8, 1e-8), (1e-30, 1e-12), (1e-8, 2.0 ** -24), (1e3, 1e-8)))
@pytest.mark.parametrize("G", (8, 16, 32, 64, 128))
def test_distance_from_the_exact_entropies(G, eps_l1, eps_log):
    # Elements of one magnitude, of many, few that are not zero, all alike but one; norms all over the approximation's range, and
    # among the last tiles below and above it (where a wavefront's tiles all take the exact way).
    S, C = ELEMENTS // 8192, 8192
    x, g = _normal((S * C // G, G), G)
    x[0::5] = torch.exp(3.0 * x[0::5])
    x[1::5] = torch.sign(x[1::5])
    x[2::5] *= (torch.rand(x[2::5].shape, device="cuda", generator=g) < 3.0 / G)
    x[3::5] = 1.0 + 0.01 * x[3::5]
    x[3::5, 0] *= 200.0
    norm = x.abs().sum(1, keepdim=True).clamp_min(1e-20)
    power = torch.empty_like(norm).uniform_(-23.9, 23.9, generator=g)
    power[-x.shape[0] // 8:] *= 1.25
    x *= torch.exp2(power) / norm
    x = x.to(torch.bfloat16)
    cfg = tahq.make_config(1, S, C, G, tahq.BF16, 3.5, eps_l1=eps_l1, eps_log=eps_log)
    off = (_approximate(cfg, x) - _exact(cfg, x)).abs()
    print(f"[case] G={G} eps_l1 {eps_l1} eps_log {eps_log}: {float(off.max()):.3g}, of {float((off > 0).float().mean()):.2f} of the tiles", flush=True)
    assert float((off > 0).float().mean()) > 0.5, "these entropies are approximate"
    assert float(off.max()) <= SLACK


@pytest.mark.parametrize("B,S,C,G,scope", ((1, 4096, 8192, 64, 0), (2, 2048, 8192, 8, 0), (2, 2048, 8192, 128, 1), (3, 2731, 4128, 32, 0)))
@pytest.mark.parametrize("share", (0.4, 0.9, 1.0))
def test_one_hot_tiles(B, S, C, G, scope, share):
    # tiles with a single element of 1 or of another power of two among zeros, whose entropies the approximation takes for zeros of
    # either sign: all tie, a little below the all-zero tiles.  Thresholds above, among and below them.
    x, g = _normal((B * S * C // G, G), 11)
    one_hot = torch.rand(x.shape[0], device="cuda", generator=g) < share
    x[one_hot] = 0.0
    sign = torch.randint(0, 2, (x.shape[0],), device="cuda", generator=g) * 2.0 - 1.0
    x[:, G // 3] = torch.where(one_hot, sign, x[:, G // 3])
    x[1::4, G // 3] *= 2.0
    x[2::4, G // 3] *= 0.125
    x[3::16] = 0.0
    x = x.to(torch.bfloat16)
    cfg = tahq.make_config(B, S, C, G, tahq.BF16, 3.5, scope=scope)
    H, exact = _approximate(cfg, x), _exact(cfg, x)
    assert float((H - exact).abs().max()) < 1e-3, "these are the entropies"
    assert not bool((H.view(torch.int32) == -2 ** 31).any()), "an entropy of -0.0f, the selection's mark of places outside a unit"
    words = -(-B * S * C // G // 64)
    for budget in (3.002, 3.0625, 3.3, 3.6, 3.93, 3.999):
        print(f"[case] one-hot [{B},{S},{C}] G={G} scope={scope} share {share} budget {budget}", flush=True)
        cfg = tahq.make_config(B, S, C, G, tahq.BF16, budget, scope=scope)
        packed = _both_ways(cfg, x)
        chosen = np.unpackbits(packed[64:64 + 8 * words].cpu().numpy(), bitorder="little").sum()
        assert int(chosen) == tahq.tahq_k_per_unit(cfg) * (1 if scope else B), "so many tiles are wide"


def test_other_constants_take_the_exact_way():
    x, _ = _normal((1, ELEMENTS // 8192, 8192), 5)
    x = x.to(torch.bfloat16)
    for eps_l1, eps_log in ((0.0, 1e-8), (1e-8, 0.0), (1e-8, 0.5), (1.0, 1e-8), (1e-3, 2.0 ** -24)):
        print(f"[case] eps_l1 {eps_l1} eps_log {eps_log}", flush=True)
        _both_ways(tahq.make_config(1, x.shape[1], 8192, 64, tahq.BF16, 3.5, eps_l1=eps_l1, eps_log=eps_log), x)
