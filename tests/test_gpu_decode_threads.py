"""Workgroups of the decode kernel that few pairs and long caches are given: weights, importance, kept set and cache are those of the workgroup
that a call without a stated bound gets, bit for bit, and the output is right."""
import ctypes

import pytest
import torch

pytestmark = pytest.mark.gpu

def threads_of(B, p, ring=False):
    rule = B.lib()._ZN3swa20decode_block_threadsERK10swa_paramslib
    bound = min(p.len_bound or p.cap, p.cap)
    return rule(ctypes.byref(p), ctypes.c_int64(p.b * p.h), bound, ctypes.c_bool(ring))


F16, BF16, F32 = torch.float16, torch.bfloat16, torch.float32
FEW = [(form, dtype, d, bound, 512) for form in ("unordered", "ordered", "two_call", "shared", "window")
       for dtype, d, bound in ((F16, 128, 257), (F32, 128, 300), (BF16, 64, 1023), (F32, 64, 1023))]
LONG = [("unordered", F16, 128, 4481, 1024), ("unordered", BF16, 64, 7168, 1024), ("unordered", F32, 64, 4700, 1024), ("unordered", F32, 128, 3585, 1024),
        ("shared", F16, 128, 3585, 1024), ("shared", BF16, 64, 3841, 1024), ("shared", F32, 128, 7168, 1024),
        ("ordered", F16, 128, 2049, 1024), ("ordered", BF16, 64, 4481, 1024), ("ordered", F32, 64, 9216, 1024), ("ordered", F32, 128, 9200, 1024),
        ("two_call", F16, 128, 8961, 1024), ("two_call", BF16, 64, 9024, 1024), ("two_call", F32, 64, 16384, 1024), ("two_call", F32, 128, 16300, 1024)]


@pytest.mark.parametrize("form,dtype,d,bound,threads", FEW + LONG)
@pytest.mark.parametrize("ahead", [1, 5])                              # most of the cache is evicted, one token
def test_stated_bound_changes_the_workgroup_and_not_the_step(form, dtype, d, bound, threads, ahead):
    from paper_2403_17312_amd import binding as B
    lens = [bound - 1, bound - 2, 200, 0] if bound < 4000 else [bound - 1, 70]
    b, h, cap, w, R = len(lens), 3, bound, 16, 8
    g = torch.Generator(device="cuda").manual_seed(37)
    flags = {"unordered": B.SWA_FUSE_COMPACTION | B.SWA_UNORDERED, "ordered": B.SWA_FUSE_COMPACTION, "two_call": 0,
             "shared": B.SWA_FUSE_COMPACTION | B.SWA_UNORDERED | B.SWA_HEAD_SHARED, "window": B.SWA_FUSE_COMPACTION | B.SWA_UNORDERED}[form]
    K0, V0 = (torch.randn((b, h, cap, d), generator=g, device="cuda").to(dtype) for _ in range(2))
    q, kn, vn = (torch.randn((b, h, d), generator=g, device="cuda").to(dtype) for _ in range(3))
    s0 = torch.rand((b, h, cap), generator=g, device="cuda")
    r0 = torch.rand((b, h, R, cap), generator=g, device="cuda")
    len0 = torch.tensor(lens, dtype=torch.int32, device="cuda")
    seq = len0 * ahead + 1 if ahead == 1 else (len0 * 5).clamp(min=1)
    got = []
    for stated in (0, bound):
        p = B.make_params(b, h, d, cap, w, 8000, dtype, len_bound=stated, flags=flags)
        assert (threads_of(B, p, form == "window") == threads) == (stated > 0)
        ws = torch.zeros(B.swa_workspace_bytes(p), dtype=torch.uint8, device="cuda")
        B.swa_workspace_init(p, ws)
        x = {"K": K0.clone(), "V": V0.clone(), "score": s0.clone(), "ring": r0.clone(), "cl": len0.clone(), "kc": torch.zeros_like(len0),
             "pos": torch.arange(cap, dtype=torch.int32, device="cuda").repeat(b, h, 1).contiguous(),
             "probs": torch.zeros((b, h, cap), device="cuda"), "kept": torch.zeros((b, h, cap), dtype=torch.int32, device="cuda"),
             "out": torch.zeros((b, h, d), device="cuda", dtype=dtype)}
        if form == "window":
            B.swa_decode_step_window(p, q, kn, vn, x["K"], x["V"], x["ring"], R, 3, x["score"], x["pos"], x["cl"], seq, x["kept"], x["kc"],
                                     x["out"], x["probs"], ws)
        else:
            B.swa_decode_step(p, q, kn, vn, x["K"], x["V"], x["score"], x["pos"], x["cl"], seq, x["kept"], x["kc"], x["out"], x["probs"], ws)
        assert B.swa_check_status(p, ws) == B.SWA_OK
        got.append(x)
    one, two = got
    for a in ("cl", "kc", "probs", "score", "pos", "K", "V", "ring"):
        assert torch.equal(one[a], two[a]), a
    # fp32 sums of at most 16384 terms (2^-20 of their magnitude), one rounding to the output type
    u = {torch.float32: 2.0 ** -20, torch.float16: 2.0 ** -11, torch.bfloat16: 2.0 ** -8}[dtype]
    for i, n in enumerate(lens):
        k = two["kc"][i].item()
        assert torch.equal(one["kept"][i, :, :k], two["kept"][i, :, :k])
        at = two["kept"][i, :, :k].long()
        rows = torch.cat([V0[i, :, :n], vn[i][:, None]], 1).double()
        pk = torch.gather(two["probs"][i].double(), 1, at)
        vk = torch.gather(rows, 1, at[..., None].expand(-1, -1, d))
        want, mag = ((pk[:, None] @ y)[:, 0] / pk.sum(1, keepdim=True) if k else torch.zeros((h, d), device="cuda", dtype=torch.float64)
                     for y in (vk, vk.abs()))
        dense = (two["probs"][i, :, :n + 1].double()[:, None] @ rows.abs())[:, 0]
        # (a few evicted rows are subtracted from the dense sum, whose magnitude then counts, over a kept mass of at least 1/20)
        assert bool(((two["out"][i].double() - want).abs() <= u * want.abs() + 2.0 ** -20 * (mag + 20 * dense)).all()), (n, k)


@pytest.mark.parametrize("dtype,d,bound,few,many,form", [
    (F16, 128, 500, 126, 129, "unordered"), (F32, 128, 300, 126, 129, "two_call"), (BF16, 64, 1023, 126, 129, "window"), (F16, 128, 300, 96, 99, "unordered"),
    (F16, 128, 3000, 255, 258, "ordered"), (F16, 128, 250, 510, 513, "unordered"), (F32, 64, 250, 510, 513, "two_call")])
def test_other_pairs_change_an_output_in_its_last_bits_only(dtype, d, bound, few, many, form):
    """The same pairs in a call of their own, which gets another workgroup or kernel, and in one with three pairs more."""
    from paper_2403_17312_amd import binding as B
    h, cap, R = 3, bound, 8
    b = many // h
    g = torch.Generator(device="cuda").manual_seed(43)
    flags = {"unordered": B.SWA_FUSE_COMPACTION | B.SWA_UNORDERED, "ordered": B.SWA_FUSE_COMPACTION, "two_call": 0,
             "window": B.SWA_FUSE_COMPACTION | B.SWA_UNORDERED}[form]
    K0, V0 = (torch.randn((b, h, cap, d), generator=g, device="cuda").to(dtype) for _ in range(2))
    q, kn, vn = (torch.randn((b, h, d), generator=g, device="cuda").to(dtype) for _ in range(3))
    s0 = torch.rand((b, h, cap), generator=g, device="cuda")
    r0 = torch.rand((b, h, R, cap), generator=g, device="cuda")
    len0 = (bound - 1 - 7 * torch.arange(b, device="cuda") % (bound // 2)).to(torch.int32)
    got, threads = [], []
    for n in (few // h, b):
        p = B.make_params(n, h, d, cap, 16, 8000, dtype, len_bound=bound, flags=flags)
        threads.append(threads_of(B, p, form == "window"))
        ws = torch.zeros(B.swa_workspace_bytes(p), dtype=torch.uint8, device="cuda")
        B.swa_workspace_init(p, ws)
        x = {"K": K0[:n].clone(), "V": V0[:n].clone(), "score": s0[:n].clone(), "ring": r0[:n].clone(), "cl": len0[:n].clone(),
             "kc": torch.zeros_like(len0[:n]), "pos": torch.arange(cap, dtype=torch.int32, device="cuda").repeat(n, h, 1).contiguous(),
             "probs": torch.zeros((n, h, cap), device="cuda"), "kept": torch.zeros((n, h, cap), dtype=torch.int32, device="cuda"),
             "out": torch.zeros((n, h, d), device="cuda", dtype=dtype)}
        seq, rows = (len0 + 1)[:n].contiguous(), (q[:n].contiguous(), kn[:n].contiguous(), vn[:n].contiguous())
        if form == "window":
            B.swa_decode_step_window(p, *rows, x["K"], x["V"], x["ring"], R, 3, x["score"], x["pos"], x["cl"], seq, x["kept"], x["kc"],
                                     x["out"], x["probs"], ws)
        else:
            B.swa_decode_step(p, *rows, x["K"], x["V"], x["score"], x["pos"], x["cl"], seq, x["kept"], x["kc"], x["out"], x["probs"], ws)
        assert B.swa_check_status(p, ws) == B.SWA_OK
        got.append(x)
    assert bound == 250 or threads[0] != threads[1]
    one, two = got
    n = few // h
    for a in ("cl", "kc", "probs", "score", "pos", "K", "V", "ring"):
        assert torch.equal(one[a], two[a][:n]), a
    # values of N(0,1) weighted by at most 1: the same fp32 terms in another order (2^-18 of their magnitude), rounded once to the output type
    u = {F32: 2.0 ** -18, F16: 2.0 ** -10, BF16: 2.0 ** -7}[dtype]
    x, y = one["out"].double(), two["out"][:n].double()
    assert bool(((x - y).abs() <= u * (y.abs() + 1.0)).all())
