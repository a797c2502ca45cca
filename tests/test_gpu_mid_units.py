"""Ranking units of 32769 to 65536 tiles against the oracle: by phases, where one workgroup ranks each from its registers, as it does in
one call of larger tensors, and in one call, which ranks those of small tensors in the quantizer's launch."""
import numpy as np
import pytest
import torch

import workloads
from oracle import o32
import paper_2506_01352_amd as tahq

pytestmark = pytest.mark.gpu

G = 8


def _encode_by_phases(cfg, d, codec):
    codec.workspace.fill_(0xFF)
    codec.packed.fill_(0xFF)
    for phase in (tahq.PHASE_PROLOGUE, tahq.PHASE_ENTROPY, tahq.PHASE_SELECT, tahq.PHASE_QUANT):
        tahq.tahq_encode_phases(cfg, d, codec.packed, codec.workspace, phase)


def _check(x, B, S, C, budget, scope=0):
    cfg = tahq.make_config(B, S, C, G, tahq.BF16, budget, scope=scope)
    codec = tahq.Codec(cfg, device="cuda")
    codec.workspace.fill_(0xFF)
    codec.packed.fill_(0xFF)
    d = torch.from_numpy(x.view(np.int16)).cuda()
    codec.encode(d)
    apart = tahq.Codec(cfg, device="cuda")
    _encode_by_phases(cfg, d, apart)
    torch.cuda.synchronize()
    want = o32.encode(o32.make_cfg(B, S, C, G, o32.BF16, budget, scope=scope), x)
    assert np.array_equal(codec.packed.cpu().numpy(), want), "stream differs from the oracle"
    assert np.array_equal(apart.packed.cpu().numpy(), want), "stream of the phases one by one differs from the oracle"


@pytest.mark.parametrize("tiles", (32769, 32832, 40001, 49152, 65473, 65474, 65535, 65536, 65537))
def test_units_of_all_lengths(tiles):
    # three samples, off the 64-tile boundaries where the length is; the last lengths that fit, by where the unit starts, and the
    # first that does not
    rng = np.random.default_rng(tiles)
    x = workloads.f32_to_bf16_bits(rng.standard_normal((3, tiles, G)).astype(np.float32)).reshape(3, tiles, G)
    for budget in (3.0 + 1.0 / tiles, 3.37, 3.9):
        print(f"[case] 3 units of {tiles} tiles, budget {budget}", flush=True)
        _check(np.ascontiguousarray(x), 3, tiles, G, float(np.float32(budget)))


@pytest.mark.parametrize("share,how", ((0.02, "zero"), (0.4, "zero"), (0.4, "constant"), (1.0, "constant"), (0.3, "one-hot"), (0.01, "nan")))
@pytest.mark.parametrize("tiles,scope", ((40000, 0), (27001, 1)))
def test_crowds_at_the_threshold(tiles, scope, share, how):
    # tiles of one entropy, more and fewer than are placed directly, with the threshold above, among and below them (3 x 27001
    # tiles as one unit, by phases: in two launches)
    rng = np.random.default_rng(int(100 * share) + tiles)
    x = rng.standard_normal((3, tiles, G)).astype(np.float32)
    at = rng.random((3, tiles)) < share
    x[at] = {"zero": np.zeros(G), "constant": np.full(G, 1.5), "one-hot": np.eye(G)[2], "nan": np.full(G, np.nan)}[how]
    x = np.ascontiguousarray(workloads.f32_to_bf16_bits(x).reshape(3, tiles, G))
    if how == "nan":                                     # (outside the contract; the two selections agree)
        d = torch.from_numpy(x.view(np.int16)).cuda()
        cfg = tahq.make_config(3, tiles, G, G, tahq.BF16, 3.5, scope=scope)
        a, b, c = (tahq.Codec(cfg, device="cuda") for _ in range(3))
        a.encode(d)
        tahq.tahq_encode_phases(cfg, d, b.packed, b.workspace, tahq.PHASE_ALL | tahq.SELECT_MULTI_LAUNCH)
        _encode_by_phases(cfg, d, c)
        torch.cuda.synchronize()
        assert torch.equal(a.packed, b.packed) and torch.equal(c.packed, b.packed)
        return
    for budget in (3.005, 3.3, 3.62, 3.85, 3.995):
        print(f"[case] {tiles} tiles, scope {scope}, {share} {how}, budget {budget}", flush=True)
        _check(x, 3, tiles, G, budget, scope)


@pytest.mark.parametrize("share", (0.0001, 0.3, 0.9, 1.0))
@pytest.mark.parametrize("tiles,scope", ((40001, 0), (27001, 1), (33000, 1)))
def test_entropies_of_all_bits_set(tiles, scope, share):
    # fp32 values of all bits set, as memory that is filled with 0xff holds, give NaN entropies of that pattern: the lowest key there is.
    # Few and many of them beside other NaN of either sign, with thresholds above, among and below them; the multi-launch selection
    # ranks by the keys' digits.
    rng = np.random.default_rng(int(100 * share) + tiles)
    B = 3 if scope == 0 else 2 if tiles == 27001 else 1
    x = rng.standard_normal((B, tiles, G)).astype(np.float32)
    bits = x.view(np.uint32)
    bits[rng.random((B, tiles)) < share] = 0xffffffff
    for pattern in (0x7fc00000, 0xfffffffe, 0xffc00001, 0x7f800000):
        bits[rng.random((B, tiles)) < 0.002, 3] = pattern
    d = torch.from_numpy(x).cuda()
    units = 1 if scope else B
    H = torch.empty(B * tiles, device="cuda")
    tahq.tahq_tile_entropy(tahq.make_config(B, tiles, G, G, tahq.F32, 3.5), d, H)
    assert bool((H.view(torch.int32) == -1).any()), "such entropies occur"
    n = B * tiles // units
    for k in (1, n // 100, n // 2, int(0.69 * n), int(0.71 * n), int(0.95 * n), n - 2, n - 1):
        cfg = tahq.make_config(B, tiles, G, G, tahq.F32, float(np.float32(3.0 + k / n)), scope=scope)
        print(f"[case] {units} units of {n} tiles, {share} with all bits set, k = {tahq.tahq_k_per_unit(cfg)}", flush=True)
        a, b = tahq.Codec(cfg, device="cuda"), tahq.Codec(cfg, device="cuda")
        for c in (a, b):
            c.workspace.fill_(0xFF)
            c.packed.fill_(0xFF)
        a.encode(d)
        tahq.tahq_encode_phases(cfg, d, b.packed, b.workspace, tahq.PHASE_ALL | tahq.SELECT_MULTI_LAUNCH)
        apart = tahq.Codec(cfg, device="cuda")
        _encode_by_phases(cfg, d, apart)
        torch.cuda.synchronize()
        assert torch.equal(a.packed, b.packed), "the two selections differ"
        assert torch.equal(apart.packed, b.packed), "the selection of the phases one by one differs"
        T = B * tiles
        chosen = np.unpackbits(a.packed[64:64 + -(-T // 64) * 8].cpu().numpy(), bitorder="little").sum()
        assert int(chosen) == units * tahq.tahq_k_per_unit(cfg)


@pytest.mark.parametrize("units", (256, 257))
def test_units_as_many_as_have_a_compute_unit_each_and_one_more(units):
    # fp32 units of 33001 tiles: ranked from registers, and in two launches
    tiles = 33001
    gen = torch.Generator(device="cuda")
    gen.manual_seed(units)
    x = torch.randn(units, tiles, G, device="cuda", generator=gen)
    x[:, ::7] = 0.0
    cfg = tahq.make_config(units, tiles, G, G, tahq.F32, 3.6)
    a, b = tahq.Codec(cfg, device="cuda"), tahq.Codec(cfg, device="cuda")
    for c in (a, b):
        c.workspace.fill_(0xFF)
        c.packed.fill_(0xFF)
    a.encode(x)
    tahq.tahq_encode_phases(cfg, x, b.packed, b.workspace, tahq.PHASE_ALL | tahq.SELECT_MULTI_LAUNCH)
    torch.cuda.synchronize()
    assert torch.equal(a.packed, b.packed), "the two selections differ"
