"""The importance seed where its keys are cut into slices (few pairs, long caches), and where the attention kernel hands
over the row statistics: every prompt length around the slices' ends, against plain fp64 attention weights."""
import ctypes
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


@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16, torch.float32])
@pytest.mark.parametrize("cap", [200, 330])                # the attention kernel for short prompts, the one for longer ones
def test_leading_keys_without_weight(dtype, cap):
    """Keys whose logits are -inf before a row's first finite logit weigh nothing: in the statistics that the attention
    kernel hands over as in the seed on its own, and in the attention output."""
    from paper_2403_17312_amd import binding as B
    b, h, d, R, dead = 2, 3, 64, 16, 40
    lens = [cap - 1, 70]
    g = torch.Generator(device="cuda").manual_seed(23)
    k, v, q = (torch.randn((b, h, cap, d), generator=g, device="cuda").to(dtype) for _ in range(3))
    k[:, :, :dead, 5] = -math.inf
    q[..., 5] = q[..., 5].abs() + 0.5
    tail = torch.stack([q[i, :, n - R:n] for i, n in enumerate(lens)]).contiguous()
    cl = torch.tensor(lens, dtype=torch.int32, device="cuda")
    p = B.make_params(b, h, d, cap, 4, 8000, dtype)
    ws = torch.zeros(B.swa_workspace_bytes(p), dtype=torch.uint8, device="cuda")
    alone, after = (torch.full((b, h, cap), float("nan"), device="cuda") for _ in range(2))
    out = torch.zeros_like(q)
    B.swa_prefill_scores(p, tail, R, k, cl, alone, ws)
    B.swa_prefill_attention(p, q, k, v, cl, out, R, after, ws)
    # weights and output rounded once each (unit roundoff u), fp32 sums
    u = {torch.float16: 2.0 ** -11, torch.bfloat16: 2.0 ** -8, torch.float32: 2.0 ** -20}[dtype]
    for i, n in enumerate(lens):
        want = torch.zeros((h, cap), device="cuda", dtype=torch.float64)
        want[:, :n] = reference(tail[i], k[i], n, R, d).sum(1)
        for got in (alone, after):
            torch.testing.assert_close(got[i].double(), want, rtol=1e-5, atol=1e-12)
        w = reference(q[i, :, :n], k[i], n, n, d)[:, dead:]
        ref, mag = w @ v[i, :, :n].double(), w @ v[i, :, :n].double().abs()
        err = (out[i, :, dead:n].double() - ref).abs()
        assert bool((err <= 1.5 * u * (mag + ref.abs()) + 1e-5).all()), f"length {n}: off by {err.max().item():.3g}"


@pytest.mark.parametrize("dtype,d,R", [(torch.float16, 128, 64), (torch.bfloat16, 64, 100), (torch.float32, 64, 16)])
@pytest.mark.parametrize("bound", [130, 257, 900, 1030, 2050])
def test_bound_below_the_capacity(dtype, d, R, bound):
    """A stated bound on the lengths places the slices; the columns behind it are cleared all the same."""
    from paper_2403_17312_amd import binding as B
    cap = 2600
    lens = [0, 1, R, bound // 2, bound - 33, bound - 2, bound - 1]
    b, h = len(lens), 2
    g = torch.Generator(device="cuda").manual_seed(17)
    q, k, v = (torch.randn((b, h, cap, d), generator=g, device="cuda").to(dtype) for _ in range(3))
    tail = torch.randn((b, h, R, d), generator=g, device="cuda").to(dtype)
    for i, n in enumerate(lens):
        for x in (q, k, v):
            x[i, :, n:] = float("nan")
        r = min(R, n)
        if n:
            tail[i, :, R - r:] = q[i, :, n - r:n]
    cl = torch.tensor(lens, dtype=torch.int32, device="cuda")
    p = B.make_params(b, h, d, cap, 4, 8000, dtype, len_bound=bound)
    ws = torch.zeros(B.swa_workspace_bytes(p), dtype=torch.uint8, device="cuda")
    alone, after = (torch.full((b, h, cap), float("nan"), device="cuda") for _ in range(2))
    B.swa_prefill_scores(p, tail, R, k, cl, alone, ws)
    B.swa_prefill_attention(p, q, k, v, cl, torch.zeros_like(q), R, after, ws)
    rows = None
    if R <= B.SWA_MAX_WINDOW_ROWS:
        rows = torch.full((b, h, R, cap), float("nan"), device="cuda")
        B.swa_prefill_rows(p, tail, R, k, cl, rows, ws)
    for i, n in enumerate(lens):
        want = torch.zeros((h, R, cap), device="cuda", dtype=torch.float64)
        if n:
            want[:, :, :n] = reference(tail[i], k[i], n, R, d)
        # as in test_slices
        for got in (alone, after):
            torch.testing.assert_close(got[i].double(), want.sum(1), rtol=1e-5, atol=1e-12)
        if rows is not None:
            torch.testing.assert_close(rows[i].double(), want, rtol=1e-5, atol=1e-12)


@pytest.mark.parametrize("dtype,d,cap,R", [(torch.float16, 128, 4200, 64), (torch.bfloat16, 64, 4200, 33),
                                           (torch.float16, 64, 2200, 32), (torch.float32, 64, 4200, 64), (torch.float32, 128, 2200, 7)])
@pytest.mark.parametrize("h", [1, 4])
def test_statistics_in_four_chains(dtype, d, cap, R, h):
    """Few pairs, the statistics' four chains in one workgroup (slices of 256 columns) and in one each (slices that can bring all
    four along): prompts that end around a round of the chains' tiles."""
    from paper_2403_17312_amd import binding as B
    lens = [R - 1, 33, 127, 128, 129, 1023, 1025, 2047, 2049, cap]
    b = len(lens)
    if dtype != torch.float32 or d == 64:                  # (rows of 512 bytes have a form of their own)
        place, apart = (getattr(B.lib(), n) for n in ("_ZN3swa16seed_stats_placeEliiiRiS0_", "_ZN3swa17seed_chains_apartEiiii"))
        place.restype, apart.restype = None, ctypes.c_bool
        G, cols = ctypes.c_int(), ctypes.c_int()
        place(ctypes.c_int64(b * h), cap, cap, R, ctypes.byref(G), ctypes.byref(cols))
        assert apart(G, cols, cap, R) is (h == 4)
    g = torch.Generator(device="cuda").manual_seed(29)
    k = torch.randn((b, h, cap, d), generator=g, device="cuda").to(dtype)
    tail = torch.randn((b, h, R, d), generator=g, device="cuda").to(dtype)
    for i, n in enumerate(lens):
        k[i, :, n:] = float("nan")
    cl = torch.tensor(lens, dtype=torch.int32, device="cuda")
    p = B.make_params(b, h, d, cap, 4, 8000, dtype)
    ws = torch.zeros(B.swa_workspace_bytes(p), dtype=torch.uint8, device="cuda")
    score = torch.full((b, h, cap), float("nan"), device="cuda")
    B.swa_prefill_scores(p, tail, R, k, cl, score, ws)
    rows = torch.full((b, h, R, cap), float("nan"), device="cuda")
    B.swa_prefill_rows(p, tail, R, k, cl, rows, ws)
    for i, n in enumerate(lens):
        want = torch.zeros((h, R, cap), device="cuda", dtype=torch.float64)
        want[:, :, :n] = reference(tail[i], k[i], n, R, d)
        # fp32 logits, exponentials and sums over at most 4200 keys and 64 rows, exponents up to about 10
        torch.testing.assert_close(score[i].double(), want.sum(1), rtol=1e-5, atol=1e-12)
        torch.testing.assert_close(rows[i].double(), want, rtol=1e-5, atol=1e-12)
