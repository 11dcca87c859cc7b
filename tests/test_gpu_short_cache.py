"""The kernel for caches of few slots against the streaming kernel, which serves the same call when no bound on the lengths is
stated: weights, importance, kept set and cache bit for bit, and the outputs of both against the sum over the kept rows in 64 bits."""
import ctypes

import pytest
import torch

pytestmark = pytest.mark.gpu

W, SPARSITY = 4, 8000                       # nint(n / 5) tokens are kept


def _evictions(m):
    """Nothing, one token, a few, half of the tokens, and most of them (whose values are read behind the selection)."""
    return 0, 1, 3, m // 2, m - m // 5


def _state(B, form, dtype, d, lens, h, cap, ties, R, g):
    """Inputs of one step: every length with every number of evictions."""
    kinds = len(_evictions(1))
    b = len(lens) * kinds
    cl = [n for n in lens for _ in range(kinds)]
    seq = [max(5 * max(n + 1 - _evictions(n + 1)[i % kinds], 1), n + 1) for i, n in enumerate(cl)]
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
    if form.startswith("window"):
        x["ring"] = torch.rand((b, h, R, cap), generator=g, device="cuda")
        if ties:
            x["ring"] = torch.floor(x["ring"] * 2)
    if form.endswith("8"):
        x["K"], x["V"] = (torch.randint(0, 256, (b, h, cap, d), generator=g, device="cuda", dtype=torch.uint8) for _ in range(2))
        x["qp"] = torch.rand((4, b, h, d), generator=g, device="cuda") * 0.02 + 0.005
        x["qp"][1::2] = torch.randint(100, 156, (2, b, h, d), generator=g, device="cuda").float()
    return b, x


def _params(B, form, dtype, d, cap, b, h, bound):
    flags = {"unordered": 3, "window": 3, "int8": 3, "window8": 3, "two_call": 0, "shared": 7, "shared8": 7}[form]
    return B.make_params(b, h, d, cap, W, SPARSITY, dtype, len_bound=bound, flags=flags | (B.SWA_KV_INT8 if form.endswith("8") else 0))


def _form(B, p, ring):
    """Threads per workgroup of the kernel for few slots, 0 where the streaming kernel serves the call."""
    rule = getattr(B.lib(), "_ZN3swa10short_formERK10swa_paramslib")
    rule.restype = ctypes.c_uint64          # {int nt, u}
    return rule(ctypes.byref(p), ctypes.c_int64(p.b * p.h), p.len_bound or p.cap, ctypes.c_bool(ring)) & 0xffffffff


def _step(B, form, dtype, d, cap, b, h, x, bound, R):
    x = {k: v.clone() for k, v in x.items()}
    p = _params(B, form, dtype, d, cap, b, h, bound)
    ws = torch.zeros(B.swa_workspace_bytes(p), dtype=torch.uint8, device="cuda")
    x["kc"] = torch.zeros_like(x["cl"])
    x["ki"] = torch.full((b, h, cap), -1, dtype=torch.int32, device="cuda")
    x["out"] = torch.zeros((b, h, d), dtype=dtype, device="cuda")
    x["probs"] = torch.full((b, h, cap), 9.0, device="cuda")
    tail = (x["score"], x["pos"], x["cl"], x["sl"], x["ki"], x["kc"], x["out"], x["probs"], ws)
    if form == "window8":
        B.swa_decode_step_window_q8(p, x["q"], x["kn"], x["vn"], x["K"], x["V"], x["qp"], x["ring"], R, R // 2, *tail)
    elif form.endswith("8"):
        B.swa_decode_step_q8(p, x["q"], x["kn"], x["vn"], x["K"], x["V"], x["qp"], *tail)
    elif form == "window":
        B.swa_decode_step_window(p, x["q"], x["kn"], x["vn"], x["K"], x["V"], x["ring"], R, R // 2, *tail)
    else:
        B.swa_decode_step(p, x["q"], x["kn"], x["vn"], x["K"], x["V"], *tail)
    assert B.swa_check_status(p, ws) == 0
    return x


def _check_outputs(form, dtype, x, before, i):
    """Sequence i's outputs against the kept rows' sum in 64 bits, from the weights and the cache that the call returned.

    Either kernel adds at most 256 terms p |v| in fp32, a lane at most 16 of them in a row and the lanes and waves in a tree, about 40
    roundings deep with the weights' own and the quotient's; where the evicted rows are subtracted the terms are all rows' and
    the divisor is the kept mass.  Then one rounding to the output type.  Codes: lambda (sum - z), with the sum formed of codes.
    """
    k, n = int(x["kc"][i]), int(before["cl"][i])          # slot n is the new token's
    at = x["ki"][i, :, :k].long()
    h, d = x["out"].shape[1:]
    v = (x["V"][i, :, :k] if form != "two_call" else x["V"][i].gather(1, at[..., None].expand(h, k, d))).double()
    w = x["probs"][i].double()[..., None]
    p = w.gather(1, at[..., None])
    mass = p.sum(1)
    new = 255.0 if form.endswith("8") else before["vn"][i].double().abs()
    peak = (before["V"][i, :, :n].double().abs() * w[:, :n]).sum(1) + new * w[:, n]
    want = (p * v).sum(1) / mass
    if form.endswith("8"):
        lam, z = x["qp"][2, i].double(), x["qp"][3, i].double()
        want, peak = lam * (want - z), lam * (peak + z)
    u = {torch.float32: 0.0, torch.float16: 2.0 ** -11, torch.bfloat16: 2.0 ** -8}[dtype]
    err = (x["out"][i].double() - want).abs()
    assert bool((err <= 40 * 2.0 ** -24 * (peak / mass + want.abs()) + u * want.abs() + 2.0 ** -24).all()), (form, i, k, n, err.max().item())


def _compare(B, form, dtype, d, lens, h, cap, bound, ties, R, g):
    b, x = _state(B, form, dtype, d, lens, h, cap, ties, R, g)
    assert _form(B, _params(B, form, dtype, d, cap, b, h, 0), R > 0) == 0
    served = dtype != torch.float32 or d != 128 or bound <= 128          # (rows of 512 bytes: 128 slots at most)
    assert (_form(B, _params(B, form, dtype, d, cap, b, h, bound), R > 0) > 0) is served
    one, two = (_step(B, form, dtype, d, cap, b, h, x, n, R) for n in (0, bound))
    assert torch.equal(one["kc"], two["kc"]) and torch.equal(one["cl"], two["cl"]) and torch.equal(one["probs"], two["probs"])
    for i in range(b):
        k = int(one["kc"][i])
        n = int(x["cl"][i]) + 1
        for a in ("score", "pos", "K", "V", "ki"):
            live = n if form == "two_call" and a != "ki" else k
            u, v = one[a][i, :, :live], two[a][i, :, :live]
            assert torch.equal(u.nan_to_num(7.0) if u.is_floating_point() else u, v.nan_to_num(7.0) if v.is_floating_point() else v), (a, i)
        if R:
            assert torch.equal(one["ring"][i, :, :, :k], two["ring"][i, :, :, :k]), i
        _check_outputs(form, dtype, one, x, i)
        _check_outputs(form, dtype, two, x, i)


@pytest.mark.parametrize("form,dtype,d,R", [
    ("unordered", torch.float16, 128, 0), ("unordered", torch.bfloat16, 128, 0), ("unordered", torch.float32, 128, 0),
    ("unordered", torch.float16, 64, 0), ("unordered", torch.bfloat16, 64, 0), ("unordered", torch.float32, 64, 0),
    ("two_call", torch.float16, 128, 0), ("two_call", torch.float32, 64, 0), ("two_call", torch.bfloat16, 64, 0),
    ("int8", torch.float16, 128, 0), ("int8", torch.float16, 64, 0),
    ("shared", torch.float16, 128, 0), ("shared", torch.bfloat16, 64, 0), ("shared", torch.float32, 64, 0),
    ("shared", torch.float32, 128, 0), ("shared8", torch.float16, 128, 0), ("shared8", torch.float16, 64, 0),
    ("window", torch.float16, 128, 1), ("window", torch.float16, 128, 33), ("window", torch.bfloat16, 64, 64),
    ("window", torch.float32, 64, 16), ("window", torch.float32, 128, 40),
    ("window8", torch.float16, 128, 16), ("window8", torch.float16, 64, 5), ("window8", torch.float16, 64, 33)])
@pytest.mark.parametrize("bound", [33, 64, 128, 192, 256])
@pytest.mark.parametrize("ties", [False, True])
def test_step_matches_the_streaming_kernel(form, dtype, d, R, bound, ties):
    from paper_2403_17312_amd import binding as B
    lens = sorted({0, 1, 5, 31, 32, bound // 2, bound - 33 if bound > 40 else 7, bound - 2, bound - 1})
    g = torch.Generator(device="cuda").manual_seed(bound * 7 + d)
    # 19 heads, more than one round of loads of their sum, and at most 512 pairs a launch, so that every form is taken
    for part in (lens[::2], lens[1::2]) if form.startswith("shared") else (lens,):
        _compare(B, form, dtype, d, part, 19 if form.startswith("shared") else 3, 611, bound, ties, R, g)


@pytest.mark.parametrize("dtype,d,bound", [(torch.float16, 64, 192), (torch.float16, 128, 190)])
def test_heads_summed_in_a_launch_of_their_own(dtype, d, bound):
    """Beyond pairs x heads x bound of 8 Mi the head-shared step has a third launch for the sum."""
    from paper_2403_17312_amd import binding as B
    lens, h = [0, 63, bound // 2, bound - 1], 56
    assert len(lens) * len(_evictions(1)) * h * h * bound > 8 << 20
    _compare(B, "shared", dtype, d, lens, h, 300, bound, False, 0, torch.Generator(device="cuda").manual_seed(3))


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
    assert _form(B, _params(B, "unordered", dtype, d, cap, b, h, 64), False) > 0
    out = _step(B, "unordered", dtype, d, cap, b, h, x, 64, 0)["out"].float()
    want = torch.zeros((b, h, d), dtype=torch.bool, device="cuda")
    want[1, :, 7] = True
    if evict == 0:
        want[0, :, 5] = True
    assert torch.equal(out.isnan(), want)
