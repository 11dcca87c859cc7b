"""The unordered step of long caches whose selection has no key array (many pairs, about 3650 to 4480 slots) against the same pairs
in calls of few, which have one: the same bits, with and without equal importance values across the line of the selection."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,d", [(torch.float16, 64), (torch.float32, 64), (torch.bfloat16, 128)])
@pytest.mark.parametrize("ties", [False, True])
@pytest.mark.parametrize("evict", [1, 40, 3000])
def test_selection_without_a_key_array(dtype, d, ties, evict):
    from paper_2403_17312_amd import binding as B
    b, h, n, cap = 48, 16, 4100, 4101
    g = torch.Generator(device="cuda").manual_seed(evict + d)
    x = {k: torch.randn((b, h, cap, d), generator=g, device="cuda").to(dtype) for k in ("K", "V")}
    x.update({k: torch.randn((b, h, d), generator=g, device="cuda").to(dtype) for k in ("q", "kn", "vn")})
    x["score"] = torch.rand((b, h, cap), generator=g, device="cuda") - 0.1          # (some below zero: the other order of bits)
    if ties:
        x["score"] = torch.floor(x["score"] * 300) / 300
        x["q"].zero_()
    x["pos"] = torch.argsort(torch.rand((b, h, cap), generator=g, device="cuda"), -1).to(torch.int32)
    x["cl"] = torch.randint(n - 200, n + 1, (b,), generator=g, device="cuda").to(torch.int32)
    x["sl"] = ((x["cl"] + 1 - evict) * 5).clamp(min=cap + 1)
    x["kc"] = torch.zeros_like(x["cl"])
    x["ki"] = torch.full((b, h, cap), -1, dtype=torch.int32, device="cuda")
    x["out"] = torch.zeros((b, h, d), dtype=dtype, device="cuda")

    def step(s):
        p = B.make_params(s["q"].shape[0], h, d, cap, 16, 8000, dtype, len_bound=cap, flags=B.SWA_FUSE_COMPACTION | B.SWA_UNORDERED)
        ws = torch.zeros(B.swa_workspace_bytes(p), dtype=torch.uint8, device="cuda")
        B.swa_decode_step(p, s["q"], s["kn"], s["vn"], s["K"], s["V"], s["score"], s["pos"], s["cl"], s["sl"], s["ki"], s["kc"],
                          s["out"], None, ws)
        assert B.swa_check_status(p, ws) == 0
        return s

    want = [step({k: v[i:i + 12].clone() for k, v in x.items()}) for i in range(0, b, 12)]
    step(x)
    for k in ("kc", "out"):
        assert torch.equal(x[k], torch.cat([w[k] for w in want])), k
    keep = x["kc"].tolist()
    assert evict < 40 or min(int(x["cl"][i]) + 1 - keep[i] for i in range(b)) > 1
    for i in range(b):
        for k in ("score", "pos", "ki", "K", "V"):
            assert torch.equal(x[k][i, :, :keep[i]], want[i // 12][k][i % 12, :, :keep[i]]), (k, i)
