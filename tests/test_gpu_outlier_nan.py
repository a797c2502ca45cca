"""The outlier test on fp32 tiles that hold NaN: a NaN counts as the smallest magnitude, and no index leaves the tile."""
import numpy as np
import pytest
import torch

from oracle import o32, o64
import paper_2506_01352_amd as tahq

pytestmark = pytest.mark.gpu

GUARD = 4096


def _encode(x, G, budget, **kw):
    """Pivot bytes, scales, zero-points, widths and payload of the stream, encoded between guard bytes."""
    B, S, C = x.shape
    cfg = tahq.make_config(B, S, C, G, tahq.F32, budget, **kw)
    size = tahq.tahq_packed_size(cfg)
    raw = torch.full((size + 2 * GUARD,), 0xA5, dtype=torch.uint8, device="cuda")
    ws = torch.full((tahq.tahq_workspace_size(cfg),), 0x3C, dtype=torch.uint8, device="cuda")
    tahq.tahq_encode(cfg, torch.from_numpy(x).cuda(), raw[GUARD:GUARD + size], ws)
    torch.cuda.synchronize()
    host = raw.cpu().numpy()
    assert (host[:GUARD] == 0xA5).all() and (host[GUARD + size:] == 0xA5).all(), "written outside the stream"
    return _sections(host[GUARD:GUARD + size], cfg)


def _sections(stream, cfg):
    T = cfg.batch * cfg.seq * cfg.hidden // cfg.tile
    off = o64.section_offsets(T, cfg.tile, cfg.batch, tahq.tahq_k_per_unit(cfg), 3)
    return (stream[off["pivot"]:][:T], stream[off["scale"]:][:2 * T].view(np.uint16), stream[off["zero"]:][:2 * T].view(np.uint16),
            np.unpackbits(stream[off["bitmap"]:off["ranks"]], bitorder="little")[:T], stream[off["payload"]:off["total"]])


def _oracle(x, G, budget, **kw):
    B, S, C = x.shape
    return _sections(o32.encode(o32.make_cfg(B, S, C, G, o32.F32, budget, **kw), x), tahq.make_config(B, S, C, G, tahq.F32, budget, **kw))


@pytest.mark.parametrize("tau,eps_ratio", ((-np.inf, 1e-8), (2.0, -1.0)))
@pytest.mark.parametrize("tiles", (211, 66003))          # several lanes per tile, and the usual number
@pytest.mark.parametrize("G", (8, 16, 32, 64, 128))
def test_tiles_of_nan_only_are_transformed_from_their_first_element(G, tiles, tau, eps_ratio):
    # thresholds that such a tile's magnitude of nothing exceeds
    rng = np.random.default_rng(G + tiles)
    x = rng.standard_normal((1, tiles, G)).astype(np.float32)
    nan = rng.random(tiles) < 0.2
    nan[:3] = nan[-3:] = True
    x[0, nan] = np.nan
    x[0, nan & (rng.random(tiles) < 0.5)] *= -1.0
    for budget in (3.0, 3.5):
        print(f"[case] G={G} {tiles} tiles tau={tau} eps_ratio={eps_ratio} budget {budget}", flush=True)
        got, want = (f(x, G, budget, tau=tau, eps_ratio=eps_ratio) for f in (_encode, _oracle))
        assert (got[0][nan] == 0x80).all()
        assert np.array_equal(got[0][~nan], want[0][~nan]), "pivot bytes of the other tiles"
        same = ~nan & (got[3] == want[3])
        assert np.array_equal(got[1][same], want[1][same]) and np.array_equal(got[2][same], want[2][same])
        if budget == 3.0:
            a, b = (s[4].reshape(tiles, -1)[~nan] for s in (got, want))
            assert np.array_equal(a, b), "payload of the other tiles"


@pytest.mark.parametrize("tiles", (211, 66003))
@pytest.mark.parametrize("G", (8, 16, 32, 64, 128))
def test_nan_of_every_kind_is_no_magnitude(G, tiles):
    # quiet and signalling NaN at every place but a tile's first (the oracle's search starts from that), beside two large elements:
    # the second largest stays what it is, and the tile is none of the outliers that a lost one makes it
    rng = np.random.default_rng(3 * G + tiles)
    x = rng.uniform(0.5, 1.5, size=(1, tiles, G)).astype(np.float32)
    at = rng.permuted(np.tile(np.arange(1, G), (tiles, 1)), axis=1)[:, :4]
    rows = np.arange(tiles)
    x[0, rows, at[:, 0]], x[0, rows, at[:, 1]] = 5.0, -4.0
    x[0, ::5, at[0, 0]] = 50.0
    bits = x.view(np.uint32)[0]
    kinds = np.array([0x7fa00000, 0xff800001, 0x7fbfffff, 0x7fc00000, 0xffffffff], np.uint32)
    bits[rows, at[:, 2]] = kinds[rng.integers(0, kinds.size, tiles)]
    some = rng.random(tiles) < 0.5
    bits[rows[some], at[some, 3]] = kinds[rng.integers(0, kinds.size, int(some.sum()))]
    for budget in (3.0, 3.5):
        print(f"[case] G={G} {tiles} tiles, budget {budget}", flush=True)
        got, want = (f(x, G, budget) for f in (_encode, _oracle))
        wrong = np.nonzero(got[0] != want[0])[0]
        assert wrong.size == 0, f"{wrong.size} pivot bytes differ, first in tile {wrong[0]}"
