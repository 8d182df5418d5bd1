"""mc_quantize at the sizes where its kernels change: tails of every length, spans that the workgroups do not share evenly, loads that
are dealt differently, and outputs beyond which the codes are stored past the caches -- every code against the definition in fp64."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("n", [2, 6, 8, 10, 254, 1022, 65536 + 2, 4 * 256 * 2048 - 2, 4 * 256 * 2048 + 6, 5 * 512 * 1024 + 10, 4 * 256 * 2048 * 3 + 258, 13 * 1024 * 1024 + 254, (32 << 20) + 4, (64 << 20) + 14])
def test_sizes(n, bits):
    import torch
    from paper_2209_06979_amd import binding as mc
    print(f"quantize {n} elements, {bits} bits", flush=True)
    g = torch.Generator(device="cuda")
    g.manual_seed(n)
    x = torch.randn(n, generator=g, device="cuda") * 30
    x[::7] = (torch.randint(-12, 13, (len(x[::7]),), generator=g, device="cuda") + 0.5) * 0.375    # quotients that are ties
    scale, qmax = 0.375, 127 if bits == 8 else 7
    got = mc.quantize(x, scale, bits)
    for b in range(0, n, 1 << 24):
        part = x[b:b + (1 << 24)]
        want = torch.round(part.double() / scale).clamp(-qmax, qmax).to(torch.int8)              # half to even
        if bits == 8:
            assert torch.equal(got[b:b + (1 << 24)], want)
        else:
            nibbles = want.to(torch.uint8) & 15
            assert torch.equal(got[b // 2:(b + (1 << 24)) // 2], nibbles[::2] | nibbles[1::2] << 4)
