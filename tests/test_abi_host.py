"""Host-side checks of the C ABI: the library loads, exports what include/tahq.h declares,
does its size arithmetic like the oracle, and rejects bad arguments before any GPU work."""
import ctypes as C
import os
import re

import numpy as np
import pytest

import workloads
from oracle import o32
import paper_2506_01352_amd as tahq
from paper_2506_01352_amd import binding

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_library_exports_every_declared_symbol():
    names = set()
    for header in sorted(os.listdir(os.path.join(ROOT, "include"))):
        text = open(os.path.join(ROOT, "include", header)).read()
        text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
        names |= set(re.findall(r"\b(tahq_[a-z0-9_]+)\s*\(", text))
    assert {"tahq_encode", "tahq_decode", "tahq_packed_size", "tahq_naive_encode", "tahq_naive_decode"} <= names
    lib = C.CDLL(tahq.library_path())
    for n in sorted(names):
        assert hasattr(lib, n), n
    # and the binding offers the same names
    for n in sorted(names):
        assert hasattr(tahq, n), n


def test_sizes_match_the_oracle_layout_on_all_configs_and_variants():
    cases = [(w.batch, w.seq, w.hidden, w.tile, w.dtype, w.budget_bits, 0, 0, 0) for w in workloads.CONFIGS]
    cases += [(3, 7, 96, 32, 0, 3.3, 0, 0, 0), (3, 7, 96, 32, 0, 3.3, 1, 0, 0), (1, 1, 128, 128, 1, 3.5, 0, 0, 0),
              (2, 5, 640, 64, 1, 3.01, 0, 0, 0)]
    # allocation tiles of several quantization tiles, up to the whole token
    cases += [(3, 7, 96, 32, 0, 3.3, 0, 96, 0), (3, 7, 96, 32, 0, 3.3, 1, 32, 0), (2, 5, 640, 64, 1, 3.4, 0, 320, 0),
              (8, 4096, 8192, 64, 1, 3.25, 0, 8192, 0), (8, 4096, 8192, 64, 1, 3.25, 0, 128, 0)]
    # tiles of 8 and 16 channels, a hidden size with 25 tiles of 64 per token
    cases += [(3, 7, 96, 8, 0, 3.3, 0, 0, 0), (2, 5, 1600, 16, 1, 3.8, 0, 0, 0), (2, 5, 1600, 64, 1, 3.8, 0, 320, 0),
              (8, 4096, 8192, 8, 1, 3.25, 0, 0, 0), (1, 3, 64, 8, 0, 2.5, 1, 32, 2)]
    # other pairs of neighbouring widths
    cases += [(3, 7, 96, 32, 0, 1.5, 0, 0, 1), (2, 5, 640, 64, 1, 7.25, 0, 0, 7), (2, 5, 640, 128, 1, 5.0, 1, 0, 4),
              (8, 4096, 8192, 64, 1, 6.5, 0, 0, 6), (3, 7, 96, 8, 0, 8.0, 0, 0, 7)]
    # the INT2/INT3 mix
    cases += [(3, 7, 96, 32, 0, 2.3, 0, 0, 2), (8, 4096, 8192, 64, 1, 2.2, 0, 0, 2), (2, 5, 640, 64, 1, 3.0, 0, 320, 2),
              (2, 5, 640, 128, 1, 2.0, 1, 0, 2), (2, 5, 640, 64, 1, 3.4, 0, 0, 3)]
    for B, S, Cc, G, dt, bud, scope, A, low in cases:
        cfg = tahq.make_config(B, S, Cc, G, dt, bud, scope=scope, alloc_tile=A, low_bits=low)
        ocfg = o32.make_cfg(B, S, Cc, G, dt, bud, scope=scope, alloc_tile=A, low_bits=low)
        assert tahq.tahq_packed_size(cfg) == o32.packed_size(ocfg) > 0
        assert tahq.tahq_k_per_unit(cfg) == o32.k_per_unit(ocfg)
        assert tahq.tahq_workspace_size(cfg) > 0


def test_defaults_and_version():
    cfg = tahq.tahq_config_default()
    assert cfg.struct_size == C.sizeof(tahq.tahq_config) == 56 and cfg.alloc_tile == 0 and cfg.low_bits == 0
    assert (cfg.tile, cfg.tau, cfg.scope) == (64, 2.0, 0)
    assert abs(cfg.budget_bits - 3.8) < 1e-6 and abs(cfg.eps_log - 1e-8) < 1e-12
    assert tahq.tahq_version() >> 16 == 1
    assert tahq.tahq_status_string(0) == "ok"
    assert "workspace" in tahq.tahq_status_string(5)


def test_invalid_configs_are_rejected_with_size_zero():
    bad = [
        dict(batch=0), dict(seq=0), dict(hidden=0), dict(hidden=100), dict(tile=4), dict(tile=48), dict(tile=256),
        dict(budget_bits=2.9), dict(budget_bits=4.1), dict(budget_bits=float("nan")), dict(dtype=2), dict(scope=2),
        dict(alloc_tile=32), dict(alloc_tile=96), dict(alloc_tile=192), dict(alloc_tile=512),
        dict(low_bits=1), dict(low_bits=4), dict(low_bits=2), dict(low_bits=2, budget_bits=3.1),
        dict(low_bits=8, budget_bits=8.5), dict(low_bits=7, budget_bits=8.1), dict(low_bits=1, budget_bits=0.9),
        dict(low_bits=2, budget_bits=1.9),
    ]
    for kw in bad:
        args = dict(batch=2, seq=4, hidden=256, tile=64, dtype=0, budget_bits=3.5)
        args.update(kw)
        cfg = tahq.make_config(**args)
        assert tahq.tahq_packed_size(cfg) == 0 and tahq.tahq_workspace_size(cfg) == 0, kw
    cfg = tahq.make_config(2, 4, 256, 64, 0, 3.5)
    cfg.struct_size = 44
    assert tahq.tahq_packed_size(cfg) == 0
    # the 48-byte layout from before alloc_tile existed is still accepted; the field is then not read
    cfg = tahq.make_config(2, 4, 256, 64, 0, 3.5, alloc_tile=96)
    assert tahq.tahq_packed_size(cfg) == 0
    cfg.struct_size = 48
    assert tahq.tahq_packed_size(cfg) == tahq.tahq_packed_size(tahq.make_config(2, 4, 256, 64, 0, 3.5)) > 0
    # ... and the 52-byte layout from before low_bits existed
    cfg = tahq.make_config(2, 4, 256, 64, 0, 3.5, alloc_tile=128, low_bits=7)
    assert tahq.tahq_packed_size(cfg) == 0
    cfg.struct_size = 52
    assert tahq.tahq_packed_size(cfg) == tahq.tahq_packed_size(tahq.make_config(2, 4, 256, 64, 0, 3.5, alloc_tile=128)) > 0


def _call_encode(cfg, d_in, d_packed, cap, d_ws, wcap):
    lib = binding._load()
    return lib.tahq_encode(C.byref(cfg), d_in, d_packed, cap, d_ws, wcap, None)


def _call_decode(cfg, d_packed, nbytes, d_out, out_dtype):
    lib = binding._load()
    return lib.tahq_decode(C.byref(cfg), d_packed, nbytes, d_out, out_dtype, None, 0, None)


def test_argument_errors_come_back_before_anything_is_enqueued():
    # Fake, never-dereferenced device addresses: every call below must fail in host validation.
    cfg = tahq.make_config(2, 4, 256, 64, 0, 3.5)
    size, ws = tahq.tahq_packed_size(cfg), tahq.tahq_workspace_size(cfg)
    A, B_, W = 0x10000, 0x20000, 0x30000
    assert _call_encode(cfg, None, B_, size, W, ws) == 1
    assert _call_encode(cfg, A, None, size, W, ws) == 1
    assert _call_encode(cfg, A, B_, size, None, ws) == 1
    assert _call_encode(cfg, A, B_, size - 1, W, ws) == 4
    assert _call_encode(cfg, A, B_, size, W, ws - 1) == 5
    assert _call_encode(cfg, A + 4, B_, size, W, ws) == 6
    assert _call_encode(cfg, A, B_ + 8, size, W, ws) == 6
    bad = tahq.make_config(2, 4, 256, 4, 0, 3.5)
    assert _call_encode(bad, A, B_, 1 << 20, W, 1 << 20) == 3
    bad = tahq.make_config(2, 4, 250, 64, 0, 3.5)
    assert _call_encode(bad, A, B_, 1 << 20, W, 1 << 20) == 2
    assert _call_decode(cfg, None, size, B_, 0) == 1
    assert _call_decode(cfg, A, size - 1, B_, 0) == 4
    assert _call_decode(cfg, A, size, B_, 2) == 2
    assert _call_decode(cfg, A, size, B_ + 2, 0) == 6
    lib = binding._load()
    assert lib.tahq_encode(None, A, B_, size, W, ws, None) == 1
    assert lib.tahq_tile_entropy(C.byref(cfg), None, B_, None) == 1
    wide = tahq.make_config(2, 4, 256, 64, 0, 3.5, alloc_tile=128)
    wws = tahq.tahq_workspace_size(wide)
    assert wws > ws
    assert lib.tahq_alloc_tile_entropy(C.byref(wide), A, B_, None, wws, None) == 1
    assert lib.tahq_alloc_tile_entropy(C.byref(wide), A, B_, W, wws - 1, None) == 5
    assert lib.tahq_alloc_tile_entropy(C.byref(wide), A, B_ + 4, W, wws, None) == 6


def test_parse_header_round_trips_an_oracle_stream():
    w, x = workloads.generate(2, batch=1, seq=4)
    ocfg = o32.make_cfg(w.batch, w.seq, w.hidden, w.tile, w.dtype, 3.25, tau=3.0)
    packed = o32.encode(ocfg, x)
    cfg = tahq.tahq_parse_header(packed[:64].tobytes())
    assert (cfg.batch, cfg.seq, cfg.hidden, cfg.tile, cfg.dtype, cfg.scope) == (1, 4, 2048, 64, 0, 0)
    assert (cfg.budget_bits, cfg.tau) == (3.25, 3.0)
    assert tahq.tahq_packed_size(cfg) == packed.size and cfg.alloc_tile == 64
    ocfg = o32.make_cfg(w.batch, w.seq, w.hidden, w.tile, w.dtype, 3.25, alloc_tile=512)
    wide = o32.encode(ocfg, x)
    cfg = tahq.tahq_parse_header(wide[:64].tobytes())
    assert cfg.alloc_tile == 512 and tahq.tahq_packed_size(cfg) == wide.size
    assert tahq.tahq_k_per_unit(cfg) == o32.k_per_unit(ocfg) == 4 and cfg.low_bits == 3
    ocfg = o32.make_cfg(w.batch, w.seq, w.hidden, w.tile, w.dtype, 2.25, low_bits=2)
    narrow = o32.encode(ocfg, x)
    cfg = tahq.tahq_parse_header(narrow[:64].tobytes())
    assert cfg.low_bits == 2 and cfg.budget_bits == 2.25 and tahq.tahq_packed_size(cfg) == narrow.size
    broken = packed[:64].copy(); broken[0] = ord("X")
    with pytest.raises(tahq.TahqError):
        tahq.tahq_parse_header(broken.tobytes())


def test_naive_codec_sizes_defaults_and_argument_errors():
    from oracle import n32
    d = tahq.tahq_naive_config_default()
    assert d.struct_size == C.sizeof(tahq.tahq_naive_config) == 28 and (d.bits, d.scale, d.dtype) == (8, 1.0, 1)
    for B, S, Cc, dt, bits, c in ((2, 3, 64, 0, 8, 1.0), (16, 2048, 5120, 1, 6, 16384.0), (1, 1, 32, 1, 2, 0.5),
                                  (3, 5, 1600, 0, 16, 3.0), (1, 7, 96, 1, 7, 1e5), (8, 4096, 8192, 1, 10, 2.0 ** 20)):
        cfg = tahq.make_naive_config(B, S, Cc, dt, bits, c)
        assert tahq.tahq_naive_packed_size(cfg) == n32.packed_size(n32.make_cfg(B, S, Cc, dt, bits, c)) > 0
    ok = dict(batch=2, seq=3, hidden=64, dtype=0, bits=8, scale=1.0)
    for kw in (dict(batch=0), dict(seq=0), dict(hidden=0), dict(hidden=48), dict(dtype=2), dict(bits=1), dict(bits=17),
               dict(scale=0.0), dict(scale=-1.0), dict(scale=float("nan")), dict(scale=float("inf"))):
        bad = dict(ok); bad.update(kw)
        assert tahq.tahq_naive_packed_size(tahq.make_naive_config(**bad)) == 0, kw
    # never-dereferenced device addresses: all of these fail in host validation
    lib = binding._load()
    cfg = tahq.make_naive_config(**ok)
    size = tahq.tahq_naive_packed_size(cfg)
    A, B_ = 0x10000, 0x20000
    assert lib.tahq_naive_encode(C.byref(cfg), None, B_, size, None) == 1
    assert lib.tahq_naive_encode(C.byref(cfg), A, None, size, None) == 1
    assert lib.tahq_naive_encode(C.byref(cfg), A, B_, size - 1, None) == 4
    assert lib.tahq_naive_encode(C.byref(cfg), A + 8, B_, size, None) == 6
    assert lib.tahq_naive_encode(None, A, B_, size, None) == 1
    assert lib.tahq_naive_decode(C.byref(cfg), A, size, None, 0, None) == 1
    assert lib.tahq_naive_decode(C.byref(cfg), A, size - 1, B_, 0, None) == 4
    assert lib.tahq_naive_decode(C.byref(cfg), A, size, B_, 2, None) == 2
    assert lib.tahq_naive_decode(C.byref(cfg), A, size, B_ + 4, 0, None) == 6
    bad = tahq.make_naive_config(**dict(ok, bits=20))
    assert lib.tahq_naive_encode(C.byref(bad), A, B_, 1 << 20, None) == 2


class _FakeDeviceTensor:
    """Just enough of a torch tensor for the binding's host-side checks (nothing is launched)."""

    def __init__(self, nbytes, esize):
        self._n, self._e = nbytes // esize, esize
        self.is_cuda = True

    def is_contiguous(self):
        return True

    def data_ptr(self):
        return 0x10000

    def numel(self):
        return self._n

    def element_size(self):
        return self._e


def test_binding_refuses_tensors_that_do_not_fit_the_configuration():
    # the C ABI carries no capacity for the activation tensors: the binding checks them before the call
    cfg = tahq.make_config(2, 4, 256, 64, tahq.BF16, 3.5)
    n = 2 * 4 * 256
    packed = _FakeDeviceTensor(tahq.tahq_packed_size(cfg), 1)
    ws = _FakeDeviceTensor(tahq.tahq_workspace_size(cfg), 1)
    with pytest.raises(ValueError, match="holds"):
        tahq.tahq_encode(cfg, _FakeDeviceTensor(2 * n - 2, 2), packed, ws, stream=0)
    with pytest.raises(ValueError, match="4-byte elements"):
        tahq.tahq_encode(cfg, _FakeDeviceTensor(4 * n, 4), packed, ws, stream=0)
    with pytest.raises(ValueError, match="holds"):
        tahq.tahq_encode_noalloc(cfg, _FakeDeviceTensor(n, 2), packed, stream=0)
    with pytest.raises(ValueError, match="holds"):
        tahq.tahq_decode(cfg, packed, _FakeDeviceTensor(2 * n, 4), tahq.F32, stream=0)
    with pytest.raises(ValueError, match="2-byte elements"):
        tahq.tahq_decode(cfg, packed, _FakeDeviceTensor(8 * n, 2), tahq.F32, stream=0)
    with pytest.raises(ValueError, match="holds"):
        tahq.tahq_tile_entropy(cfg, _FakeDeviceTensor(2 * n, 2), _FakeDeviceTensor(4 * (n // 64) - 4, 4), stream=0)
    ncfg = tahq.make_naive_config(2, 4, 256, tahq.F32, 8, 4.0)
    with pytest.raises(ValueError, match="holds"):
        tahq.tahq_naive_encode(ncfg, _FakeDeviceTensor(4 * n - 4, 4), _FakeDeviceTensor(1 << 20, 1), stream=0)
    with pytest.raises(ValueError, match="holds"):
        tahq.tahq_naive_decode(ncfg, _FakeDeviceTensor(1 << 20, 1), _FakeDeviceTensor(n, 2), tahq.BF16, stream=0)


def test_more_than_65535_ranking_units_on_the_multi_launch_selection_are_refused():
    # that selection puts the ranking unit into the grid's second dimension (units large enough to take it by
    # default cannot be that many: the tensor would exceed 2^31 tiles)
    cfg = tahq.make_config(70000, 1, 256, 64, tahq.BF16, 3.5)
    lib = binding._load()
    big = 1 << 40
    assert lib.tahq_encode_phases(C.byref(cfg), 0x10000, 0x20000, big, 0x30000, big, 15 | 16, None) == 3
    cfg = tahq.make_config(65535, 1, 256, 64, tahq.BF16, 3.5)
    assert tahq.tahq_packed_size(cfg) > 0


def test_more_than_65535_ranking_units_off_the_64_tile_boundaries_are_taken():
    # 65536 units of 32706 .. 32767 tiles are the most tiles that a unit can have in a tensor of that many
    torch = pytest.importorskip("torch")
    if torch.cuda.device_count() > 0:
        pytest.skip("the addresses are made up: a call that passes the checks must find no device")
    lib = binding._load()
    big = 1 << 42
    for seq in (32705, 32706, 32767):
        cfg = tahq.make_config(65536, seq, 8, 8, tahq.BF16, 3.5)
        assert tahq.tahq_packed_size(cfg) > 0
        assert lib.tahq_encode(C.byref(cfg), 0x10000, 0x20000, big, 0x30000, big, None) == 7       # the launch fails
        assert lib.tahq_encode_phases(C.byref(cfg), 0x10000, 0x20000, big, 0x30000, big, 15 | 16, None) == 3
