"""The quantizer that works by wavefronts, at the ends of their groups of tiles, against the oracle."""
import numpy as np
import pytest
import torch

import workloads
from oracle import o32
import paper_2506_01352_amd as tahq

pytestmark = pytest.mark.gpu


def _check(B, n, G, f32, budget, low=0, seed=0):
    rng = np.random.default_rng(seed + n)
    x = rng.standard_normal((B, n, G)).astype(np.float32)
    x.reshape(-1)[rng.integers(0, x.size, x.size // 50 + 1)] *= 30.0         # outlier tiles, some at d = 0
    if not f32:
        x = workloads.f32_to_bf16_bits(x).reshape(B, n, G)
    print(f"[case] {B} units of {n} tiles of {G}, fp32 {f32}, budget {budget}", flush=True)
    cfg = tahq.make_config(B, n, G, G, tahq.F32 if f32 else tahq.BF16, budget, low_bits=low)
    codec = tahq.Codec(cfg, device="cuda")
    codec.workspace.fill_(0xFF)
    codec.packed.fill_(0xFF)
    codec.encode(torch.from_numpy(x if f32 else x.view(np.int16)).cuda())
    torch.cuda.synchronize()
    want = o32.encode(o32.make_cfg(B, n, G, G, o32.F32 if f32 else o32.BF16, budget, low_bits=low), x)
    assert np.array_equal(codec.packed.cpu().numpy(), want), "stream differs from the oracle"


@pytest.mark.parametrize("f32", (False, True))
@pytest.mark.parametrize("G", (8, 16, 32, 64, 128))
def test_one_width_in_tensors_of_few_tiles(G, f32):
    for n in (1, 15, 16, 17, 31, 33, 63, 64, 65, 127, 129, 257):
        for budget in (3.0, 4.0):
            _check(1, n, G, f32, budget)


@pytest.mark.parametrize("G,n,f32", ((8, 65537, False), (8, 65537, True), (16, 65599, False), (16, 65537, True), (32, 65537, True), (64, 32769, True),
                                     (128, 32799, False), (128, 32769, True)))
def test_one_width_in_tensors_of_more(G, n, f32):
    _check(1, n, G, f32, 3.0)
    _check(1, n, G, f32, 3.0, low=2)


@pytest.mark.parametrize("G,B,n,f32", ((8, 9, 29127, False), (16, 9, 29127, True), (32, 5, 26217, True), (64, 5, 26217, True), (128, 5, 13111, False),
                                       (128, 5, 13111, True)))
def test_two_widths(G, B, n, f32):
    # more tiles than are ranked where they are quantized, units off the boundaries of 64 tiles
    _check(B, n, G, f32, 3.3)
