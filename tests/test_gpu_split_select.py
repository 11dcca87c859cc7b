"""The split-rows step's own selection launch: kept sets and importance against the one-workgroup kernel bit for bit,
with many equal keys, budgets at the edges, lengths around the threads' runs, and both forms of the output pass."""
import ctypes

import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,d,cap", [(torch.float16, 128, 2200), (torch.float32, 64, 4099), (torch.bfloat16, 64, 16384),
                                         (torch.float32, 128, 9000)])
@pytest.mark.parametrize("w,sparsity", [(0, 9999), (7, 0), (64, 5000), (-1, 8000), (3000, 9000)])
@pytest.mark.parametrize("scores", ["spread", "ties"])
def test_selection_matches_the_one_workgroup_kernel(dtype, d, cap, w, sparsity, scores):
    from paper_2403_17312_amd import binding as B
    lens = [0, 1, 1023, 1024, 2047, cap - 2, cap - 1, cap]            # the last one is full: skipped and reported
    b, h = len(lens), 3
    g = torch.Generator(device="cuda").manual_seed(3)
    K, V = (torch.randn((b, h, cap, d), generator=g, device="cuda").to(dtype) for _ in range(2))
    q, kn, vn = (torch.randn((b, h, d), generator=g, device="cuda").to(dtype) for _ in range(3))
    old = torch.rand((b, h, cap), generator=g, device="cuda")
    if scores == "ties":
        old = torch.floor(old * 3)
        q.zero_()                                                      # equal weights: importance ties everywhere
    got = []
    for flags in (0, B.SWA_SPLIT_ROWS):
        p = B.make_params(b, h, d, cap, w, sparsity, dtype, flags=flags)
        st = B.DecodeState(p, debug_probs=True)
        st.K.copy_(K)
        st.V.copy_(V)
        st.score.copy_(old)
        st.cache_len.copy_(torch.tensor(lens, dtype=torch.int32))
        st.seq_len.copy_(torch.tensor([n + 1 for n in lens], dtype=torch.int32))
        st.decode_step(q, kn, vn)
        assert st.check_status() == B.SWA_ERR_CAPACITY
        got.append(st)
    one, two = got
    assert one.cache_len.tolist() == two.cache_len.tolist() and one.kept_cnt.tolist() == two.kept_cnt.tolist()
    u = {torch.float32: 2.0 ** -20, torch.float16: 2.0 ** -10, torch.bfloat16: 2.0 ** -7}[dtype]
    for i, n in enumerate(lens[:-1]):
        k = one.kept_cnt[i].item()
        assert torch.equal(one.score[i, :, :n + 1], two.score[i, :, :n + 1]), n
        assert torch.equal(one.probs[i], two.probs[i]), n
        assert torch.equal(one.kept_idx[i, :, :k], two.kept_idx[i, :, :k]), n
        for a in ("K", "V", "pos"):
            assert torch.equal(getattr(one, a)[i, :, :n + 1], getattr(two, a)[i, :, :n + 1]), (n, a)
        # the same fp32 terms added in another order, rounded once to the output type
        x, y = one.out[i].double(), two.out[i].double()
        assert bool(((x - y).abs() <= u * (y.abs() + 1.0)).all()), n
    assert torch.equal(one.out[-1], two.out[-1]) and torch.equal(two.score[-1], old[-1])


@pytest.mark.parametrize("dtype", [torch.float16, torch.bfloat16, torch.float32])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("w,sparsity,ahead", [(64, 8000, 1), (64, 8000, 5), (1500, 9500, 1), (0, 9999, 1), (0, 9000, 3)])
def test_output_whatever_is_kept(dtype, d, w, sparsity, ahead):
    """A cache of a much longer sequence (nearly everything is kept), a wide window, and budgets of a few rows: the launch
    that forms the output, with a number of pairs that is no multiple of the XCDs."""
    check_output(dtype, d, 5, [2499, 2049], 2500, w, sparsity, ahead)


@pytest.mark.parametrize("dtype,d", [(torch.float16, 64), (torch.float16, 128), (torch.float32, 128)])      # one, two and four pieces a row
@pytest.mark.parametrize("b,h", [(5, 13), (3, 41), (2, 64)])
@pytest.mark.parametrize("w,sparsity,ahead", [(64, 8000, 1), (64, 8000, 5), (0, 9999, 1)])
def test_output_of_more_than_64_pairs(dtype, d, b, h, w, sparsity, ahead):
    """The launch that forms the output, in pieces of 128 bytes."""
    check_output(dtype, d, h, [2199, 2049, 2198, 900, 2100][:b], 2200, w, sparsity, ahead)


def check_output(dtype, d, h, lens, cap, w, sparsity, ahead):
    from paper_2403_17312_amd import binding as B
    b = len(lens)
    pieces = B.lib()._ZN3swa17split_piece_bytesEl
    assert pieces(ctypes.c_int64(b * h)) == (64 if b * h <= 64 else 128)
    g = torch.Generator(device="cuda").manual_seed(13)
    K, V = (torch.randn((b, h, cap, d), generator=g, device="cuda").to(dtype) for _ in range(2))
    q, kn, vn = (torch.randn((b, h, d), generator=g, device="cuda").to(dtype) for _ in range(3))
    old = torch.rand((b, h, cap), generator=g, device="cuda")
    p = B.make_params(b, h, d, cap, w, sparsity, dtype, flags=B.SWA_SPLIT_ROWS)
    st = B.DecodeState(p, debug_probs=True)
    st.K.copy_(K)
    st.V.copy_(V)
    st.score.copy_(old)
    st.cache_len.copy_(torch.tensor(lens, dtype=torch.int32))
    st.seq_len.copy_(torch.tensor([ahead * (n + 1) for n in lens], dtype=torch.int32))
    st.decode_step(q, kn, vn)
    assert st.check_status() == B.SWA_OK
    u = {torch.float32: 2.0 ** -20, torch.float16: 2.0 ** -11, torch.bfloat16: 2.0 ** -8}[dtype]
    for i, n in enumerate(lens):
        k = B.swa_budget(ahead * (n + 1), n + 1, w, sparsity)[0]
        assert st.kept_cnt[i].item() == k
        at = st.kept_idx[i, :, :k].long()
        rows = torch.cat([V[i, :, :n], vn[i][:, None]], 1).double()
        pk = torch.gather(st.probs[i].double(), 1, at)
        vk = torch.gather(rows, 1, at[..., None].expand(-1, -1, d))
        want, mag = ((pk[:, None] @ x)[:, 0] / pk.sum(1, keepdim=True) if k else torch.zeros((h, d), device="cuda", dtype=torch.float64)
                     for x in (vk, vk.abs()))
        # fp32 sums of at most 2500 terms (2^-20 of their magnitude), one rounding to the output type
        assert bool(((st.out[i].double() - want).abs() <= u * want.abs() + 2.0 ** -20 * mag).all()), (n, k)


@pytest.mark.parametrize("special", ["inf", "nan", "-nan", "-inf", "huge", "negative", "-0", "tiny"])
@pytest.mark.parametrize("w,sparsity", [(0, 9000), (64, 5000)])
def test_importance_of_any_value(special, w, sparsity):
    """The range of the keys comes from the old importance where that bounds the new, and is looked for where a value is not finite."""
    import struct

    from paper_2403_17312_amd import binding as B
    b, h, d, cap = 2, 4, 64, 4200
    lens = [4199, 2500]
    g = torch.Generator(device="cuda").manual_seed(29)
    K, V = (torch.randn((b, h, cap, d), generator=g, device="cuda").half() for _ in range(2))
    q, kn, vn = (torch.randn((b, h, d), generator=g, device="cuda").half() for _ in range(3))
    old = torch.rand((b, h, cap), generator=g, device="cuda") ** 4
    at = torch.rand((b, h, cap), generator=g, device="cuda") < 0.05
    if special == "negative":
        old = torch.where(at, -old, old)
    elif special == "tiny":
        old *= 1e-38                                       # (denormals among them)
    else:
        bits = {"inf": 0x7f800000, "nan": 0x7fc00000, "-nan": 0xffc00000, "-inf": 0xff800000, "huge": 0x7f7fffff, "-0": 0x80000000}[special]
        word = struct.unpack("<i", struct.pack("<I", bits))[0]
        old = torch.where(at, torch.full_like(old, 0).view(torch.int32).fill_(word).view(torch.float32), old)
    got = []
    for flags in (0, B.SWA_SPLIT_ROWS):
        p = B.make_params(b, h, d, cap, w, sparsity, torch.float16, flags=flags)
        st = B.DecodeState(p, debug_probs=True)
        st.K.copy_(K)
        st.V.copy_(V)
        st.score.copy_(old)
        st.cache_len.copy_(torch.tensor(lens, dtype=torch.int32))
        st.seq_len.copy_(torch.tensor([n + 1 for n in lens], dtype=torch.int32))
        st.decode_step(q, kn, vn)
        assert st.check_status() == B.SWA_OK
        got.append(st)
    one, two = got
    assert one.kept_cnt.tolist() == two.kept_cnt.tolist()
    for i, n in enumerate(lens):
        k = one.kept_cnt[i].item()
        assert torch.equal(one.score[i, :, :n + 1].view(torch.int32), two.score[i, :, :n + 1].view(torch.int32)), n
        assert torch.equal(one.kept_idx[i, :, :k], two.kept_idx[i, :, :k]), n


@pytest.mark.parametrize("dtype,d,b,h,cap", [(torch.float16, 128, 4, 8, 1024), (torch.float32, 64, 4, 3, 1100), (torch.bfloat16, 128, 4, 16, 1536),
                                             (torch.float32, 128, 4, 5, 2047)])
@pytest.mark.parametrize("w,sparsity", [(0, 9999), (7, 0), (64, 8000), (900, 9000)])
def test_caches_below_2048_slots(dtype, d, b, h, cap, w, sparsity):
    """Few pairs with wide rows are split from 1024 or 1536 slots on, under a stated bound: weights, importance and kept set of the one-workgroup
    kernel."""
    from paper_2403_17312_amd import binding as B
    rule = B.lib()._ZN3swa12split_factorElibi
    assert rule(ctypes.c_int64(b * h), cap, ctypes.c_bool(True), d * (4 if dtype == torch.float32 else 2)) > 1
    lens = [cap - 1, cap - 2, 700, 0]
    g = torch.Generator(device="cuda").manual_seed(41)
    K, V = (torch.randn((b, h, cap, d), generator=g, device="cuda").to(dtype) for _ in range(2))
    q, kn, vn = (torch.randn((b, h, d), generator=g, device="cuda").to(dtype) for _ in range(3))
    old = torch.floor(torch.rand((b, h, cap), generator=g, device="cuda") * 300) / 300                # (some of them equal)
    got = []
    for flags in (0, B.SWA_SPLIT_ROWS):
        st = B.DecodeState(B.make_params(b, h, d, cap, w, sparsity, dtype, len_bound=cap, flags=flags), debug_probs=True)
        st.K.copy_(K)
        st.V.copy_(V)
        st.score.copy_(old)
        st.cache_len.copy_(torch.tensor(lens, dtype=torch.int32))
        st.seq_len.copy_(torch.tensor([n + 1 for n in lens], dtype=torch.int32))
        st.decode_step(q, kn, vn)
        assert st.check_status() == B.SWA_OK
        got.append(st)
    one, two = got
    assert one.cache_len.tolist() == two.cache_len.tolist() and one.kept_cnt.tolist() == two.kept_cnt.tolist()
    u = {torch.float32: 2.0 ** -20, torch.float16: 2.0 ** -10, torch.bfloat16: 2.0 ** -7}[dtype]
    for i, n in enumerate(lens):
        k = one.kept_cnt[i].item()
        assert torch.equal(one.score[i, :, :n + 1], two.score[i, :, :n + 1]), n
        assert torch.equal(one.probs[i], two.probs[i]), n
        assert torch.equal(one.kept_idx[i, :, :k], two.kept_idx[i, :, :k]), n
        # the same fp32 terms added in another order, rounded once to the output type
        x, y = one.out[i].double(), two.out[i].double()
        assert bool(((x - y).abs() <= u * (y.abs() + 1.0)).all()), n
