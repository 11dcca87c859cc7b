"""The importance seed where its keys are cut into slices (few pairs, long caches), and where the attention kernel hands
over the row statistics: every prompt length around the slices' ends, against plain fp64 attention weights."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu


def reference(q, k, n, R, d):
    """[h, R, n] attention weights of the last R prompt queries (zeros for rows before the prompt)."""
    z = q.double() @ k[:, :n].double().transpose(1, 2).contiguous() / math.sqrt(d)
    t = torch.arange(n - R, n, device="cuda")[:, None]
    z = z.masked_fill(torch.arange(n, device="cuda")[None, :] > t, -math.inf)
    return torch.where(t >= 0, torch.softmax(z, -1), torch.zeros_like(z))


@pytest.mark.parametrize("dtype,d,cap,R", [(torch.float16, 128, 2100, 64), (torch.bfloat16, 64, 1024, 128),
                                           (torch.float32, 64, 1311, 33), (torch.float16, 64, 1025, 1)])
def test_slices(dtype, d, cap, R):
    from paper_2403_17312_amd import binding as B
    lens = [0, 1, R, 255, 256, 257, 511, 513, cap // 2 + 1, cap - 1, cap]
    b, h = len(lens), 2
    g = torch.Generator(device="cuda").manual_seed(11)
    k, v = (torch.randn((b, h, cap, d), generator=g, device="cuda").to(dtype) for _ in range(2))
    q = torch.randn((b, h, cap, d), generator=g, device="cuda").to(dtype)
    tail = torch.randn((b, h, R, d), generator=g, device="cuda").to(dtype)
    for i, n in enumerate(lens):
        k[i, :, n:] = float("nan")
        v[i, :, n:] = float("nan")
        q[i, :, n:] = float("nan")
        if n:
            r = min(R, n)
            tail[i, :, R - r:] = q[i, :, n - r:n]
    cl = torch.tensor(lens, dtype=torch.int32, device="cuda")
    p = B.make_params(b, h, d, cap, 4, 8000, dtype)
    ws = torch.zeros(B.swa_workspace_bytes(p), dtype=torch.uint8, device="cuda")
    alone = torch.full((b, h, cap), float("nan"), device="cuda")
    B.swa_prefill_scores(p, tail, R, k, cl, alone, ws)
    after = torch.full((b, h, cap), float("nan"), device="cuda")
    B.swa_prefill_attention(p, q, k, v, cl, torch.zeros_like(q), R, after, ws)
    rows = None
    if R <= B.SWA_MAX_WINDOW_ROWS:
        rows = torch.full((b, h, R, cap), float("nan"), device="cuda")
        B.swa_prefill_rows(p, tail, R, k, cl, rows, ws)
    for i, n in enumerate(lens):
        want = torch.zeros((h, R, cap), device="cuda", dtype=torch.float64)
        if n:
            want[:, :, :n] = reference(tail[i], k[i], n, R, d)
        # fp32 logits, exponentials and sums over at most 2100 keys and 128 rows, exponents up to about 10
        for got in (alone, after):
            torch.testing.assert_close(got[i].double(), want.sum(1), rtol=1e-5, atol=1e-12)
        if rows is not None:
            torch.testing.assert_close(rows[i].double(), want, rtol=1e-5, atol=1e-12)
