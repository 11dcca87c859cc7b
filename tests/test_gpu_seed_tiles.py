"""The importance seed's key tiles at every prompt length around the ends of tiles and of the four waves' rounds, and the sums of many
keys, which are read past the caches, against plain fp64 attention weights."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu

LENS = sorted({max(0, 32 * n + e) for n in range(0, 14) for e in (-1, 0, 1)})


def rows_of(q, k, n, R, d):
    """[h, R, n] attention weights of the last R prompt queries (zeros for rows before the prompt)."""
    z = q.double() @ k[:, :n].double().transpose(1, 2).contiguous() / math.sqrt(d)
    t = torch.arange(n - R, n, device="cuda")[:, None]
    z = z.masked_fill(torch.arange(n, device="cuda")[None, :] > t, -math.inf)
    return torch.where(t >= 0, torch.softmax(z, -1), torch.zeros_like(z))


@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
@pytest.mark.parametrize("d,R", [(128, 1), (128, 32), (64, 33), (128, 64), (64, 97)])
def test_every_tile_count(dtype, d, R):
    from paper_2403_17312_amd import binding as B
    b, h, cap = len(LENS), 2, max(LENS) + 3
    g = torch.Generator(device="cuda").manual_seed(31)
    k = torch.randn((b, h, cap, d), generator=g, device="cuda").to(dtype)
    tail = torch.randn((b, h, R, d), generator=g, device="cuda").to(dtype)
    for i, n in enumerate(LENS):
        k[i, :, n:] = float("nan")                        # rows past a prompt must not be used
    cl = torch.tensor(LENS, dtype=torch.int32, device="cuda")
    p = B.make_params(b, h, d, cap, 4, 8000, dtype)
    ws = torch.zeros(B.swa_workspace_bytes(p), dtype=torch.uint8, device="cuda")
    score = torch.full((b, h, cap), float("nan"), device="cuda")
    B.swa_prefill_scores(p, tail, R, k, cl, score, ws)
    ring = None
    if R <= B.SWA_MAX_WINDOW_ROWS:
        ring = torch.full((b, h, R, cap), float("nan"), device="cuda")
        B.swa_prefill_rows(p, tail, R, k, cl, ring, ws)
    for i, n in enumerate(LENS):
        want = torch.zeros((h, R, cap), device="cuda", dtype=torch.float64)
        if n:
            want[:, :, :n] = rows_of(tail[i], k[i], n, R, d)
        # fp32 logits, exponentials and sums over at most 417 keys and 97 rows, exponents up to about 10
        torch.testing.assert_close(score[i].double(), want.sum(1), rtol=1e-5, atol=1e-12)
        if ring is not None:
            torch.testing.assert_close(ring[i].double(), want, rtol=1e-5, atol=1e-12)


@pytest.mark.parametrize("R", [16, 64])
def test_sums_of_more_keys_than_the_caches_hold(R):
    """More than 128 MB of keys: the sums after the attention read them past the caches; same bits as one sequence at a time."""
    from paper_2403_17312_amd import binding as B
    b, h, d, cap = 33, 16, 128, 1100
    lens = [cap - 31 * i for i in range(b)]
    g = torch.Generator(device="cuda").manual_seed(32)
    q, k, v = (torch.randn((b, h, cap, d), generator=g, device="cuda").half() for _ in range(3))
    cl = torch.tensor(lens, dtype=torch.int32, device="cuda")
    ws = torch.zeros(1024, dtype=torch.uint8, device="cuda")
    many, one = (torch.full((b, h, cap), float("nan"), device="cuda") for _ in range(2))
    out = torch.zeros_like(q)
    B.swa_prefill_attention(B.make_params(b, h, d, cap, 4, 8000, torch.float16), q, k, v, cl, out, R, many, ws)
    p = B.make_params(1, h, d, cap, 4, 8000, torch.float16)
    for i in range(b):
        B.swa_prefill_attention(p, q[i:i + 1], k[i:i + 1], v[i:i + 1], cl[i:i + 1], out[i:i + 1], R, one[i:i + 1], ws)
    assert torch.equal(many, one)
