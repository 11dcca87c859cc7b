"""Prefill attention in the 16-bit formats at every number of key tiles around the rotation of its three LDS buffers,
and at lengths around the ends of tiles and query blocks, against plain fp64 attention."""
import math

import pytest
import torch

pytestmark = pytest.mark.gpu

LENS = sorted({max(1, 32 * n + e) for n in range(0, 11) for e in (-1, 0, 1)} | {255, 257, 385})


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
def test_every_tile_count(dtype, d):
    from paper_2403_17312_amd import binding as B
    b, h, cap = len(LENS), 3, max(LENS) + 5
    g = torch.Generator(device="cuda").manual_seed(5)
    q, k, v = (torch.randn((b, h, cap, d), generator=g, device="cuda").to(dtype) for _ in range(3))
    lens = torch.tensor(LENS, dtype=torch.int32, device="cuda")
    beyond = torch.arange(cap, device="cuda")[None, None, :, None] >= lens[:, None, None, None]
    for x in (q, k, v):
        x.masked_fill_(beyond, float("nan"))          # rows past a prompt must not be used
    out = torch.full_like(q, 7.0)
    p = B.make_params(b, h, d, cap, 4, 8000, dtype)
    ws = torch.zeros(B.swa_workspace_bytes(p), dtype=torch.uint8, device="cuda")
    B.swa_prefill_attention(p, q, k, v, lens, out, 0, None, ws)
    # weights are rounded once to the cache type before the second product and the output once (unit roundoff u),
    # sums are fp32: |delta_c| <= 1.5 u (sum_j p_j |v_jc| + |out_c|) + 1e-5
    u = 2.0 ** -11 if dtype == torch.float16 else 2.0 ** -8
    for i, n in enumerate(LENS):
        Q, K, V = (x[i, :, :n].double() for x in (q, k, v))
        z = Q @ K.transpose(1, 2).contiguous() / math.sqrt(d)
        z = z.masked_fill(torch.ones(n, n, device="cuda", dtype=torch.bool).triu(1), -math.inf)
        pr = torch.softmax(z, -1)
        ref, mag = pr @ V, pr @ V.abs()
        err = (out[i, :, :n].double() - ref).abs()
        assert bool((err <= 1.5 * u * (mag + ref.abs()) + 1e-5).all()), f"length {n}: off by {err.max().item():.3g}"
        assert bool((out[i, :, n:] == 7.0).all()), f"length {n}: wrote past the prompt"


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16])
@pytest.mark.parametrize("cap,bound,R", [(256, 0, 0), (256, 0, 64), (256, 0, 128), (255, 0, 128), (250, 0, 1), (390, 256, 100),
                                         (390, 256, 128), (390, 257, 128), (390, 255, 128), (64, 0, 33), (64, 0, 32)])
def test_either_side_of_the_short_prompt_line(dtype, d, cap, bound, R):
    """The kernel for short prompts (bound of at most 256 rows) and the other one just above: outputs, and the importance seed
    from statistics that the attention kernel hands over (2 R up to the bound) or that the seed forms itself."""
    from paper_2403_17312_amd import binding as B
    top = min(cap, bound - 1) if bound else cap
    lens = sorted({n for n in (0, 1, 2, 31, 32, 33, 63, 64, 65, 127, 128, 129, 160, 254, 255, 256, top - 1, top) if n <= top})
    b, h = len(lens), 3
    g = torch.Generator(device="cuda").manual_seed(6)
    q, k, v = (torch.randn((b, h, cap, d), generator=g, device="cuda").to(dtype) for _ in range(3))
    cl = torch.tensor(lens, dtype=torch.int32, device="cuda")
    beyond = torch.arange(cap, device="cuda")[None, None, :, None] >= cl[:, None, None, None]
    for x in (q, k, v):
        x.masked_fill_(beyond, float("nan"))          # rows past a prompt must not be used
    out = torch.full_like(q, 7.0)
    score = torch.full((b, h, cap), float("nan"), device="cuda") if R else None
    p = B.make_params(b, h, d, cap, 4, 8000, dtype, len_bound=bound)
    ws = torch.zeros(B.swa_workspace_bytes(p), dtype=torch.uint8, device="cuda")
    B.swa_prefill_attention(p, q, k, v, cl, out, R, score, ws)
    u = 2.0 ** -11 if dtype == torch.float16 else 2.0 ** -8          # as in test_every_tile_count
    for i, n in enumerate(lens):
        Q, K, V = (x[i, :, :n].double() for x in (q, k, v))
        z = Q @ K.transpose(1, 2).contiguous() / math.sqrt(d)
        z = z.masked_fill(torch.ones(n, n, device="cuda", dtype=torch.bool).triu(1), -math.inf)
        pr = torch.softmax(z, -1)
        ref, mag = pr @ V, pr @ V.abs()
        err = (out[i, :, :n].double() - ref).abs()
        assert bool((err <= 1.5 * u * (mag + ref.abs()) + 1e-5).all()), f"length {n}: off by {err.max().item():.3g}"
        assert bool((out[i, :, n:] == 7.0).all()), f"length {n}: wrote past the prompt"
        if R:
            # fp32 logits, exponentials and sums over at most 256 keys and 128 rows, exponents up to about 10
            torch.testing.assert_close(score[i, :, :n].double(), pr[:, max(0, n - R):].sum(1), rtol=1e-5, atol=1e-12)
            assert bool((score[i, :, n:] == 0.0).all()), f"length {n}: score beyond the prompt"


@pytest.mark.parametrize("dtype,d", [(torch.float16, 128), (torch.bfloat16, 64), (torch.float32, 64)])
@pytest.mark.parametrize("b,h,bound", [(61, 7, 400), (1, 5, 700), (9, 1, 1100), (131, 8, 129)])
def test_every_query_block_is_dealt_out_once(dtype, d, b, h, bound):
    """Pairs dealt out one after the other, block by block, and both in one launch, against launches of one sequence each."""
    from paper_2403_17312_amd import binding as B
    g = torch.Generator(device="cuda").manual_seed(8)
    lens = [(i * 37) % (bound + 1) for i in range(b - 1)] + [bound]
    q, k, v = (torch.randn((b, h, bound, d), generator=g, device="cuda").to(dtype) for _ in range(3))
    cl = torch.tensor(lens, dtype=torch.int32, device="cuda")
    ws = torch.zeros(1024, dtype=torch.uint8, device="cuda")
    got, one = torch.full_like(q, 7.0), torch.full_like(q, 7.0)
    B.swa_prefill_attention(B.make_params(b, h, d, bound, 4, 8000, dtype), q, k, v, cl, got, 0, None, ws)
    p = B.make_params(1, h, d, bound, 4, 8000, dtype)
    for i in range(b):
        B.swa_prefill_attention(p, q[i:i + 1], k[i:i + 1], v[i:i + 1], cl[i:i + 1], one[i:i + 1], 0, None, ws)
    assert torch.equal(got, one)


@pytest.mark.parametrize("dtype,d", [(torch.float16, 128), (torch.bfloat16, 64), (torch.float32, 64)])
@pytest.mark.parametrize("bound", [100, 128, 300])
def test_rows_below_a_bound_that_a_prompt_exceeds(dtype, d, bound):
    """A prompt longer than the stated bound: the rows below the bound are those of the same call without one."""
    from paper_2403_17312_amd import binding as B
    b, h, cap = 4, 3, 700
    g = torch.Generator(device="cuda").manual_seed(9)
    q, k, v = (torch.randn((b, h, cap, d), generator=g, device="cuda").to(dtype) for _ in range(3))
    lens = [bound - 1, bound, bound + 61, cap]
    cl = torch.tensor(lens, dtype=torch.int32, device="cuda")
    ws = torch.zeros(1024, dtype=torch.uint8, device="cuda")
    got, want = torch.full_like(q, 7.0), torch.full_like(q, 7.0)
    B.swa_prefill_attention(B.make_params(b, h, d, cap, 4, 8000, dtype, len_bound=bound), q, k, v, cl, got, 0, None, ws)
    B.swa_prefill_attention(B.make_params(b, h, d, cap, 4, 8000, dtype), q, k, v, cl, want, 0, None, ws)
    # two kernels where one side is served by the one for short prompts: each within 1.5 u (sum_j p_j |v_jc| + |out_c|) + 1e-5 of the
    # exact result (test_every_tile_count), and both terms are at most max |v| < 7
    u = {torch.float16: 2.0 ** -11, torch.bfloat16: 2.0 ** -8, torch.float32: 2.0 ** -20}[dtype]
    for i, n in enumerate(lens):
        top = min(n, bound)
        err = (got[i, :, :top].float() - want[i, :, :top].float()).abs().max().item()
        assert err <= 2 * (1.5 * u * 2 * 7 + 1e-5), (n, err)
