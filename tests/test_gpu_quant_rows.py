"""KV compression around the number of rows a workgroup keeps in registers, for every workgroup size, against the formulas
of the compression in plain fp32 (one IEEE rounding per operation): parameters and codes bit for bit."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("cap,lens", [(576, [0, 1, 31, 32, 33, 511, 512, 513, 576]), (1280, [1, 63, 577, 1023, 1024, 1025, 1280]),
                                      (2200, [5, 127, 129, 2047, 2048, 2049, 2200])])
def test_rows(d, cap, lens):
    from paper_2403_17312_amd import binding as B
    b, h = len(lens), 3
    g = torch.Generator(device="cuda").manual_seed(9)
    K, V = (torch.randn((b, h, cap, d), generator=g, device="cuda").half() for _ in range(2))
    V[..., 0] = 0.25                                    # a flat channel
    V[..., 1] *= 8000.0            # a wide one (normal values stay below 8 in size: 64000 < 65504, the largest fp16)
    K[..., 2] *= 2.0 ** -18                             # a range below 2^-7, subnormal values
    for i, n in enumerate(lens):
        K[i, :, n:] = float("nan")
        V[i, :, n:] = float("nan")
    cl = torch.tensor(lens, dtype=torch.int32, device="cuda")
    p = B.make_params(b, h, d, cap, 4, 8000, torch.float16)
    cK, cV = (torch.full((b, h, cap, d), 7, dtype=torch.uint8, device="cuda") for _ in range(2))
    qp = torch.full((4, b, h, d), float("nan"), device="cuda")
    B.swa_quantize_kv(p, K, V, cl, cK, cV, qp)
    for i, n in enumerate(lens):
        for x, codes, at in ((K, cK, 0), (V, cV, 2)):
            f = x[i, :, :n].float()
            lo = f.amin(1) if n else torch.zeros((h, d), device="cuda")
            hi = f.amax(1) if n else torch.zeros((h, d), device="cuda")
            lam = (hi - lo).clamp(min=2.0 ** -7) / torch.full((h, d), 255.0, device="cuda")
            z = torch.round(-lo / lam)
            assert torch.equal(qp[at, i], lam) and torch.equal(qp[at + 1, i], z), (n, at)
            want = torch.round(f / lam[:, None] + z[:, None]).clamp(0, 255).to(torch.uint8)
            assert torch.equal(codes[i, :, :n], want), (n, at)
            assert bool((codes[i, :, n:] == 7).all()), (n, at)


@pytest.mark.parametrize("stated", [False, True])
@pytest.mark.parametrize("d,h,cap,lens", [(64, 62, 64, [0, 1, 63, 64, 17]), (64, 62, 576, [0, 3, 111, 112, 113, 575, 576, 200, 40]),
                                          (128, 150, 1280, [1280, 0, 255, 256, 257, 1024]), (128, 150, 1280, [200, 31, 256]), (64, 400, 1280, [300, 1024, 16, 384]), (64, 700, 1280, [300, 1024, 16, 256]),
                                          (64, 130, 2200, [16, 2200, 447, 448, 449, 1500]), (64, 130, 2200, [448, 0])])
def test_short_and_longer_prompts_side_by_side(d, h, cap, lens, stated):
    """More pieces than the chip holds at once: the kernel for short prompts and the one for longer ones divide the pairs
    among them, with one workgroup per piece (a stated bound) or with a narrow grid, which may find nothing to do."""
    from paper_2403_17312_amd import binding as B
    b = len(lens)
    g = torch.Generator(device="cuda").manual_seed(31)
    K, V = (torch.randn((b, h, cap, d), generator=g, device="cuda", dtype=torch.float16) for _ in range(2))
    for i, n in enumerate(lens):
        K[i, :, n:] = float("nan")
        V[i, :, n:] = float("nan")
    cl = torch.tensor(lens, dtype=torch.int32, device="cuda")
    p = B.make_params(b, h, d, cap, 4, 8000, torch.float16, len_bound=max(lens) + 1 if stated else 0)
    cK, cV = (torch.full((b, h, cap, d), 7, dtype=torch.uint8, device="cuda") for _ in range(2))
    qp = torch.full((4, b, h, d), float("nan"), device="cuda")
    B.swa_quantize_kv(p, K, V, cl, cK, cV, qp)
    for i, n in enumerate(lens):
        for x, codes, at in ((K, cK, 0), (V, cV, 2)):
            f = x[i, :, :n].float()
            lo = f.amin(1) if n else torch.zeros((h, d), device="cuda")
            hi = f.amax(1) if n else torch.zeros((h, d), device="cuda")
            lam = (hi - lo).clamp(min=2.0 ** -7) / torch.full((h, d), 255.0, device="cuda")
            z = torch.round(-lo / lam)
            assert torch.equal(qp[at, i], lam) and torch.equal(qp[at + 1, i], z), (n, at)
            want = torch.round(f / lam[:, None] + z[:, None]).clamp(0, 255).to(torch.uint8)
            assert torch.equal(codes[i, :, :n], want), (n, at)
            assert bool((codes[i, :, n:] == 7).all()), (n, at)
