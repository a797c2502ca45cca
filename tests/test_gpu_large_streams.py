"""Streams so large that their payload is stored past the caches: the bytes of the samples' own streams, which are not."""
import pytest
import torch

from oracle import o64
import paper_2506_01352_amd as tahq

pytestmark = pytest.mark.gpu

PAST_THE_CACHES = 112 << 20
B = 9


@pytest.mark.parametrize("budget", (3.25, 3.0, 4.0))     # ranked, and one width of either kind
@pytest.mark.parametrize("G,dtype", ((8, tahq.BF16), (16, tahq.BF16), (32, tahq.BF16), (64, tahq.BF16), (128, tahq.BF16),
                                     (32, tahq.F32), (128, tahq.F32)))
def test_the_same_bytes_as_sample_by_sample(G, dtype, budget):
    # payload units of one to sixteen bytes; samples of whole words of the bit map, so that the sections are the samples' one after
    # the other, and an odd number of words, so that the tensor ends inside a quantizer's batch
    M = 65
    S = 64 * (1 + PAST_THE_CACHES // int(B * M * (G / 8 * budget + 5.1) * 64) // 2 * 2)
    S += 128 if tahq.tahq_packed_size(tahq.make_config(B, S, M * G, G, dtype, budget)) < PAST_THE_CACHES else 0
    cfg, one = (tahq.make_config(b, S, M * G, G, dtype, budget) for b in (B, 1))
    size, n, k = tahq.tahq_packed_size(cfg), S * M, tahq.tahq_k_per_unit(one)
    assert size >= PAST_THE_CACHES > tahq.tahq_packed_size(one) and n % 128 == 64
    print(f"[case] [{B},{S},{M * G}] G={G} dtype {dtype} {budget} bits: {size / (1 << 20):.0f} MiB", flush=True)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(G)
    x = torch.empty(B, S, M * G, device="cuda", dtype=torch.bfloat16 if dtype == tahq.BF16 else torch.float32)
    for b in range(B):
        x[b] = torch.randn(S, M * G, device="cuda", generator=gen)
    x[:, :, ::997] *= 20.0
    whole, sample = tahq.Codec(cfg, device="cuda"), tahq.Codec(one, device="cuda")
    whole.packed.fill_(0xFF)
    whole.encode(x)
    whole.decode()
    all_, off = o64.section_offsets(B * n, G, B, k), o64.section_offsets(n, G, 1, k)
    payload = G // 8 * (3 * n + k)
    for b in range(B):
        sample.packed.fill_(0xFF)
        sample.encode(x[b])
        sample.decode()
        torch.cuda.synchronize()
        for name, length in (("bitmap", n // 8), ("pivot", n), ("scale", 2 * n), ("zero", 2 * n), ("payload", payload)):
            got = whole.packed[all_[name] + b * length:all_[name] + (b + 1) * length]
            assert torch.equal(got, sample.packed[off[name]:off[name] + length]), f"{name} of sample {b}"
        ranks = whole.packed[all_["ranks"] + n // 16 * b:all_["ranks"] + n // 16 * (b + 1)].view(torch.int32)
        assert torch.equal(ranks, sample.packed[off["ranks"]:off["ranks"] + n // 16].view(torch.int32) + b * k)
        assert torch.equal(whole.out.view(B, -1)[b], sample.out.view(-1)), f"decoded sample {b}"
    assert all_["payload"] + B * payload == size
