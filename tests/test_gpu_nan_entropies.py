"""Entropies of tiles with NaN of several kinds: the same whichever kernel computes them, so that all selections rank alike."""
import numpy as np
import pytest
import torch

import paper_2506_01352_amd as tahq

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", (tahq.F32, tahq.BF16))
@pytest.mark.parametrize("G", (8, 16, 32, 64, 128))
# units that the phases one by one rank by one workgroup, from its registers, in two launches (the one call ranks most of them in the
# quantizer's launch), and (bf16) of approximate entropies
@pytest.mark.parametrize("B,tiles,scope", ((3, 1024, 0), (2, 40960, 1), (3, 77700, 0), (1, 98304, 0), (1, 0, 0)))
def test_tiles_of_any_bits(B, tiles, scope, G, dtype):
    if tiles == 0:
        tiles = (1 << 25) // G
        if dtype == tahq.F32:
            pytest.skip("entropies of fp32 tensors are exact whatever their size")
    rng = np.random.default_rng(G + tiles)
    bits = rng.integers(0, 1 << (16 if dtype else 32), size=(B * tiles, G), dtype=np.uint16 if dtype else np.uint32)
    d = torch.from_numpy(bits.view(np.int16 if dtype else np.int32)).cuda()
    H = torch.empty(B * tiles, device="cuda")
    tahq.tahq_tile_entropy(tahq.make_config(B, tiles, G, G, dtype, 3.5), d, H)
    magnitude = (bits.astype(np.uint32) << 16 if dtype else bits) & np.uint32(0x7fffffff)
    most = magnitude.max(axis=1)
    nan = most > 0x7f800000
    assert nan.any()
    got = H.cpu().numpy().view(np.uint32)
    assert np.array_equal(got[nan], most[nan] | np.uint32(0x80400000)), "the largest payload, quiet, the sign turned over"
    for budget in (3.03, 3.5, 3.97):
        print(f"[case] {B} x {tiles} tiles of {G}, dtype {dtype}, scope {scope}, budget {budget}", flush=True)
        cfg = tahq.make_config(B, tiles, G, G, dtype, budget, scope=scope)
        a, b = tahq.Codec(cfg, device="cuda"), tahq.Codec(cfg, device="cuda")
        for c in (a, b):
            c.workspace.fill_(0xFF)
            c.packed.fill_(0xFF)
        a.encode(d)
        tahq.tahq_encode_phases(cfg, d, b.packed, b.workspace, tahq.PHASE_ALL | tahq.SELECT_MULTI_LAUNCH)
        torch.cuda.synchronize()
        assert torch.equal(a.packed, b.packed), "the two selections differ"
        a.packed.fill_(0xFF)
        a.workspace.fill_(0xFF)
        for phase in (tahq.PHASE_PROLOGUE, tahq.PHASE_ENTROPY, tahq.PHASE_SELECT, tahq.PHASE_QUANT):
            tahq.tahq_encode_phases(cfg, d, a.packed, a.workspace, phase)
        torch.cuda.synchronize()
        assert torch.equal(a.packed, b.packed), "the selection of the phases one by one differs"
