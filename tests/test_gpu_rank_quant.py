"""Small tensors, whose units are ranked by the quantizer's launch: byte for byte the oracle's stream, and that of the phases apart."""
import numpy as np
import pytest
import torch

import workloads
from oracle import o32
import paper_2506_01352_amd as tahq

pytestmark = pytest.mark.gpu


def _check(x, B, S, C, G, budget, low=0, scope=0, nan=False):
    f32 = x.dtype == np.float32
    cfg = tahq.make_config(B, S, C, G, tahq.F32 if f32 else tahq.BF16, budget, scope=scope, low_bits=low)
    d = torch.from_numpy(x if f32 else x.view(np.int16)).cuda()
    a, b = tahq.Codec(cfg, device="cuda"), tahq.Codec(cfg, device="cuda")
    for c in (a, b):
        c.workspace.fill_(0xFF)
        c.packed.fill_(0xFF)
    a.encode(d)
    for phase in (tahq.PHASE_PROLOGUE, tahq.PHASE_ENTROPY, tahq.PHASE_SELECT, tahq.PHASE_QUANT):
        tahq.tahq_encode_phases(cfg, d, b.packed, b.workspace, phase)
    torch.cuda.synchronize()
    got = a.packed.cpu().numpy()
    assert np.array_equal(got, b.packed.cpu().numpy()), "one launch and the phases apart differ"
    if nan:
        return                                           # (outside the contract: the two selections agree)
    want = o32.encode(o32.make_cfg(B, S, C, G, o32.F32 if f32 else o32.BF16, budget, scope=scope, low_bits=low), x)
    assert np.array_equal(got, want), "stream differs from the oracle"


def _values(rng, shape, f32):
    x = rng.standard_normal(shape).astype(np.float32)
    x.reshape(-1)[rng.integers(0, x.size, x.size // 100)] *= 40.0          # outlier tiles
    return x if f32 else workloads.f32_to_bf16_bits(x).reshape(shape)


@pytest.mark.parametrize("f32", (False, True))
@pytest.mark.parametrize("G", (8, 16, 32, 64, 128))
def test_batches_and_units_of_all_lengths(G, f32):
    # one tile to several batches per unit, on and off the 64-tile boundaries; units of one batch, of a batch and one tile, and
    # of as many as there are workgroups in one round, and one more
    rng = np.random.default_rng(G)
    most = {8: 1024, 16: 512}.get(G, 256)
    for B, n in ((1, 2), (3, 63), (2, 64), (5, 65), (3, 129), (1, most), (7, most + 1), (255, 64), (256, 64), (257, 64), (200, 67)):
        x = np.ascontiguousarray(_values(rng, (B, n, G), f32))
        for budget in (3.0 + 1.0 / n, 3.8):
            print(f"[case] {B} units of {n} tiles of {G}, fp32 {f32}, budget {budget}", flush=True)
            _check(x, B, n, G, G, float(np.float32(budget)))


@pytest.mark.parametrize("n,B", ((28672, 1), (28673, 1), (28609, 2), (28610, 2), (16383, 4), (16384, 4), (65537, 2), (86016, 2), (86017, 2), (85953, 2), (85954, 2), (98304, 1),
                                 (98305, 1), (98241, 2), (98242, 2)))
def test_the_largest_units(n, B):
    rng = np.random.default_rng(n)
    x = np.ascontiguousarray(_values(rng, (B, n, 8), False))
    for budget in (3.0 + 1.0 / n, 3.5, 4.0 - 1.0 / n):
        print(f"[case] {B} units of {n} tiles, budget {budget}", flush=True)
        _check(x, B, n, 8, 8, float(np.float32(budget)))


@pytest.mark.parametrize("G,n,B,f32", ((64, 17500, 4, False), (64, 17500, 4, True), (64, 16384, 8, True), (32, 25600, 5, True), (32, 40001, 2, False),
                                       (16, 33333, 4, True), (16, 77700, 3, False), (64, 50001, 1, True), (128, 30000, 1, False), (128, 12287, 1, True),
                                       (128, 12288, 1, True), (128, 20480, 2, True), (128, 20481, 2, True), (128, 32769, 1, True), (128, 40960, 1, True),
                                       (128, 40961, 1, True), (64, 23001, 3, True), (64, 40960, 2, True)))
def test_as_many_tiles_as_fit_one_round(G, n, B, f32):
    # lanes of more elements, entropies in LDS and from memory; the smaller thresholds' bins hold hundreds of tiles; fp32 lanes of 128
    # bytes on both sides of the lines between which they are taken
    x = np.ascontiguousarray(_values(np.random.default_rng(n), (B, n, G), f32))
    for budget in (3.07, 3.5, 3.8):
        print(f"[case] {B} units of {n} tiles of {G}, fp32 {f32}, budget {budget}", flush=True)
        _check(x, B, n, G, G, budget)


@pytest.mark.parametrize("n,values", ((30000, 3), (90000, 40), (20000, 300)))
def test_tiles_of_a_few_entropies(n, values):
    # a bin of more tiles than are listed, or than are placed directly, of a few entropies each; the threshold among, above and
    # below every one of them
    rng = np.random.default_rng(values)
    kinds = rng.standard_normal((values, 8)).astype(np.float32)
    kinds[1:] = kinds[0] + 1e-3 * kinds[1:]              # nearly alike
    x = kinds[rng.integers(0, values, (1, n))]
    for share in (1 / n, 0.11, 0.33, 0.34, 0.5, 0.75, 0.97):
        print(f"[case] {n} tiles of {values} kinds, share {share}", flush=True)
        _check(np.ascontiguousarray(x), 1, n, 8, 8, float(np.float32(3.0 + share)))


@pytest.mark.parametrize("low", (1, 2, 4, 5, 6, 7))
def test_other_widths(low):
    rng = np.random.default_rng(low)
    for G, f32 in ((8, False), (16, True), (32, False), (64, True), (128, False)):
        print(f"[case] widths {low}, {low + 1}, tiles of {G}", flush=True)
        _check(np.ascontiguousarray(_values(rng, (3, 301, G), f32)), 3, 301, G, G, low + 0.4, low=low)


@pytest.mark.parametrize("share,how", ((0.02, "zero"), (0.4, "zero"), (0.4, "constant"), (1.0, "constant"), (0.3, "one-hot"), (0.01, "nan")))
@pytest.mark.parametrize("n,scope", ((5001, 0), (8000, 1), (32001, 0)))
def test_crowds_at_the_threshold(n, scope, share, how):
    # tiles of one entropy, more and fewer than are placed directly, with the threshold above, among and below them, in units
    # of many batches
    rng = np.random.default_rng(int(100 * share) + n)
    G = 16
    x = rng.standard_normal((3, n, G)).astype(np.float32)
    x[rng.random((3, n)) < share] = {"zero": np.zeros(G), "constant": np.full(G, 1.5), "one-hot": np.eye(G)[2], "nan": np.full(G, np.nan)}[how]
    x = np.ascontiguousarray(workloads.f32_to_bf16_bits(x).reshape(3, n, G))
    for budget in (3.005, 3.3, 3.62, 3.85, 3.995):
        print(f"[case] {n} tiles, scope {scope}, {share} {how}, budget {budget}", flush=True)
        _check(x, 3, n, G, G, budget, scope=scope, nan=how == "nan")


def test_pivots_at_every_place():
    # the swap crosses the lanes of a tile: the largest element at every index of it
    for G in (8, 16, 32, 64, 128):
        x = np.random.default_rng(G).uniform(0.1, 1.0, (1, G, G)).astype(np.float32)
        x[0, np.arange(G), np.arange(G)] = -50.0
        print(f"[case] pivots of tiles of {G}", flush=True)
        _check(x, 1, G, G, G, 3.5)
        _check(np.ascontiguousarray(workloads.f32_to_bf16_bits(x).reshape(x.shape)), 1, G, G, G, 3.5)
