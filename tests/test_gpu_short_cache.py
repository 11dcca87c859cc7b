"""The kernel for caches of few slots against the streaming kernel, which serves the same call when no bound on the lengths is
stated: weights, importance, kept set and cache bit for bit, the output to the rounding of its sums."""
import pytest
import torch

pytestmark = pytest.mark.gpu

W, SPARSITY = 4, 8000                       # nint(n / 5) tokens are kept


def _state(B, form, dtype, d, lens, cap, ties, R, g):
    """Inputs of one step: every length with nothing, one token, a few and half of the tokens to evict."""
    h = 19 if form == "shared" else 3
    b = len(lens) * 4
    cl = [n for n in lens for _ in range(4)]
    seq = []
    for i, n in enumerate(cl):
        m = n + 1
        evict = (0, 1, 3, m // 2)[i % 4]
        seq.append(5 * max(m - evict, 1))
    x = {"cl": torch.tensor(cl, dtype=torch.int32, device="cuda"), "sl": torch.tensor(seq, dtype=torch.int32, device="cuda")}
    x["K"], x["V"] = (torch.randn((b, h, cap, d), generator=g, device="cuda").to(dtype) for _ in range(2))
    x["q"], x["kn"], x["vn"] = (torch.randn((b, h, d), generator=g, device="cuda").to(dtype) for _ in range(3))
    x["score"] = torch.rand((b, h, cap), generator=g, device="cuda")
    if ties:
        x["score"] = torch.floor(x["score"] * 3)
        x["q"].zero_()
    x["pos"] = torch.full((b, h, cap), -1, dtype=torch.int32, device="cuda")
    for i, n in enumerate(cl):              # distinct earlier positions; in any order where the form allows it
        same = torch.randperm(max(seq[i] - 1, n), generator=g, device="cuda")[:n].to(torch.int32)
        for j in range(h):
            at = same if form.startswith("shared") else torch.randperm(max(seq[i] - 1, n), generator=g, device="cuda")[:n].to(torch.int32)
            x["pos"][i, j, :n] = at if form != "two_call" else at.sort().values
        x["K"][i, :, n:] = float("nan")     # behind the cache: never used
        x["V"][i, :, n:] = float("nan")
    if form == "window":
        x["ring"] = torch.rand((b, h, R, cap), generator=g, device="cuda")
        if ties:
            x["ring"] = torch.floor(x["ring"] * 2)
    if form.endswith("8"):
        x["K"], x["V"] = (torch.randint(0, 256, (b, h, cap, d), generator=g, device="cuda", dtype=torch.uint8) for _ in range(2))
        x["qp"] = torch.rand((4, b, h, d), generator=g, device="cuda") * 0.02 + 0.005
        x["qp"][1::2] = torch.randint(100, 156, (2, b, h, d), generator=g, device="cuda").float()
    return b, h, x


def _step(B, form, dtype, d, cap, b, h, x, bound, R):
    x = {k: v.clone() for k, v in x.items()}
    flags = {"unordered": 3, "window": 3, "int8": 3 | B.SWA_KV_INT8, "two_call": 0, "shared": 7,
             "shared8": 7 | B.SWA_KV_INT8}[form]
    p = B.make_params(b, h, d, cap, W, SPARSITY, dtype, len_bound=bound, flags=flags)
    ws = torch.zeros(B.swa_workspace_bytes(p), dtype=torch.uint8, device="cuda")
    x["kc"] = torch.zeros_like(x["cl"])
    x["ki"] = torch.full((b, h, cap), -1, dtype=torch.int32, device="cuda")
    x["out"] = torch.zeros((b, h, d), dtype=dtype, device="cuda")
    x["probs"] = torch.full((b, h, cap), 9.0, device="cuda")
    tail = (x["score"], x["pos"], x["cl"], x["sl"], x["ki"], x["kc"], x["out"], x["probs"], ws)
    if form.endswith("8"):
        B.swa_decode_step_q8(p, x["q"], x["kn"], x["vn"], x["K"], x["V"], x["qp"], *tail)
    elif form == "window":
        B.swa_decode_step_window(p, x["q"], x["kn"], x["vn"], x["K"], x["V"], x["ring"], R, R // 2, *tail)
    else:
        B.swa_decode_step(p, x["q"], x["kn"], x["vn"], x["K"], x["V"], *tail)
    assert B.swa_check_status(p, ws) == 0
    return x


@pytest.mark.parametrize("form,dtype,d,R", [
    ("unordered", torch.float16, 128, 0), ("unordered", torch.bfloat16, 128, 0), ("unordered", torch.float32, 128, 0),
    ("unordered", torch.float16, 64, 0), ("unordered", torch.bfloat16, 64, 0), ("unordered", torch.float32, 64, 0),
    ("two_call", torch.float16, 128, 0), ("two_call", torch.float32, 64, 0), ("two_call", torch.bfloat16, 64, 0),
    ("int8", torch.float16, 128, 0), ("int8", torch.float16, 64, 0),
    ("shared", torch.float16, 128, 0), ("shared", torch.bfloat16, 64, 0), ("shared", torch.float32, 64, 0),
    ("shared", torch.float32, 128, 0), ("shared8", torch.float16, 128, 0), ("shared8", torch.float16, 64, 0),
    ("window", torch.float16, 128, 1), ("window", torch.float16, 128, 33), ("window", torch.bfloat16, 64, 64),
    ("window", torch.float32, 64, 16), ("window", torch.float32, 128, 40)])
@pytest.mark.parametrize("bound", [33, 64, 128, 192, 256])
@pytest.mark.parametrize("ties", [False, True])
def test_step_matches_the_streaming_kernel(form, dtype, d, R, bound, ties):
    from paper_2403_17312_amd import binding as B
    cap = 611
    lens = sorted({0, 1, 5, 31, 32, bound // 2, bound - 33 if bound > 40 else 7, bound - 2, bound - 1})
    g = torch.Generator(device="cuda").manual_seed(bound * 7 + d)
    b, h, x = _state(B, form, dtype, d, lens, cap, ties, R, g)          # (19 heads: more than one round of loads of their sum)
    one, two = (_step(B, form, dtype, d, cap, b, h, x, n, R) for n in (0, bound))
    assert torch.equal(one["kc"], two["kc"]) and torch.equal(one["cl"], two["cl"]) and torch.equal(one["probs"], two["probs"])
    for i in range(b):
        k = int(one["kc"][i])
        n = int(x["cl"][i]) + 1
        for a in ("score", "pos", "K", "V", "ki"):
            live = n if form == "two_call" and a != "ki" else k
            u, v = one[a][i, :, :live], two[a][i, :, :live]
            assert torch.equal(u.nan_to_num(7.0) if u.is_floating_point() else u, v.nan_to_num(7.0) if v.is_floating_point() else v), (a, i)
        if form == "window":
            assert torch.equal(one["ring"][i, :, :, :k], two["ring"][i, :, :, :k]), i
    # at most 256 fp32 terms of weight 1 in all, added in another order (256 x 2^-24), the evicted ones subtracted or left out
    # (a kept mass of at least 0.05 where they are subtracted), rounded once to the output type
    # (codes: lambda (sum - z), values up to 256 times lambda <= 0.025)
    u = {torch.float32: 2.0 ** -24, torch.float16: 2.0 ** -10, torch.bfloat16: 2.0 ** -7}[dtype]
    y, z = one["out"].double(), two["out"].double()
    peak = 7.0
    assert bool(((y - z).abs() <= u * (y.abs() + 2.0 ** -10) + 256 * 2.0 ** -24 * peak * 20).all())


def test_a_cache_beyond_the_stated_bound_is_skipped_and_reported():
    from paper_2403_17312_amd import binding as B
    b, h, d, cap = 3, 2, 128, 300
    p = B.make_params(b, h, d, cap, 4, 8000, torch.float16, len_bound=60, flags=3)
    st = B.DecodeState(p)
    st.cache_len.copy_(torch.tensor([20, 64, 299], dtype=torch.int32))
    st.seq_len.copy_(torch.tensor([100, 400, 400], dtype=torch.int32))
    st.pos.copy_(torch.arange(cap, dtype=torch.int32, device="cuda").repeat(b, h, 1))
    st.out.fill_(7.0)
    q = torch.randn((b, h, d), device="cuda").half()
    before = st.score.clone()
    st.decode_compact_step(q, q, q)
    assert st.check_status() == B.SWA_ERR_CAPACITY and st.cache_len.tolist()[1:] == [64, 299]
    assert bool((st.out[1:] == 7.0).all()) and not bool((st.out[0] == 7.0).any()) and torch.equal(st.score[1:], before[1:])


@pytest.mark.parametrize("dtype", [torch.float16, torch.float32])
@pytest.mark.parametrize("evict", [0, 1, 3])
def test_a_kept_row_counts_although_its_weight_underflows(dtype, evict):
    """0 x inf of a kept value row is NaN as in the sum over the kept rows; what an evicted row holds does not matter."""
    from paper_2403_17312_amd import binding as B
    b, h, d, cap, n = 2, 3, 128, 300, 60
    x = {"cl": torch.tensor([n, n], dtype=torch.int32, device="cuda"),
         "sl": torch.tensor([5 * (n + 1 - evict)] * 2, dtype=torch.int32, device="cuda")}
    g = torch.Generator(device="cuda").manual_seed(evict)
    x["K"], x["V"] = (torch.randn((b, h, cap, d), generator=g, device="cuda").to(dtype) for _ in range(2))
    x["kn"], x["vn"] = (torch.randn((b, h, d), generator=g, device="cuda").to(dtype) for _ in range(2))
    x["q"] = torch.ones((b, h, d), dtype=dtype, device="cuda")
    x["score"] = torch.ones((b, h, cap), device="cuda")
    x["score"][..., :evict] = 0.0                                   # these go
    x["pos"] = torch.arange(cap, dtype=torch.int32, device="cuda").repeat(b, h, 1).contiguous()
    x["K"][:, :, [0, 20]] = -30.0                                   # logits 340 below the others: weight 0
    x["V"][0, :, 0, 5] = float("inf")                               # (evicted, if anything is)
    x["V"][1, :, 20, 7] = float("inf")                              # kept
    out = _step(B, "unordered", dtype, d, cap, b, h, x, 64, 0)["out"].float()
    want = torch.zeros((b, h, d), dtype=torch.bool, device="cuda")
    want[1, :, 7] = True
    if evict == 0:
        want[0, :, 5] = True
    assert torch.equal(out.isnan(), want)
