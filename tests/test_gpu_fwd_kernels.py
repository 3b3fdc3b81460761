"""The two kernels of the bf16 forward (four waves per 64-row query tile, or
one) give the same bytes, the edge paths of the one-wave kernel meet the oracle,
and it is not given lists of which one may be far longer than the others.

Every case of the edges is a launch of 6144 tiles (six on every SIMD of 256
CUs), which the rule gives to the one-wave kernel; the same heads computed alone
are launches of 8 or 16, which take the four-wave one."""
import numpy as np
import pytest
import torch

import bench
import oracle as O
import paper_2609_23153_amd as sa
import workloads as W
from gpu_helpers import check_out, widen

pytestmark = pytest.mark.gpu

DEV = "cuda:0"
TAU = W.softmax_scale(128)
CUS = 256
# The row sum is over probabilities rounded to bf16, each within a relative
# 2^-8 of its value, so the sum is too, also where one of them is most of it;
# 1e-4 more covers the fp32 scores (up to about 500, of 128 products).
LSE_ABS = float(np.log1p(2.0 ** -8)) + 1e-4


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    sa.library()
    assert torch.cuda.get_device_properties(0).multi_processor_count == CUS
    yield
    torch.cuda.synchronize()


def one_wave(tiles, kmax, nb, block=64):
    """The launch goes to the one-wave kernel."""
    return bench.forward_kernel(tiles, kmax, nb, block, CUS) == "fwd_bf16_wave_kernel"


def make_lists(kind, B, H, nb, kmax, seed):
    """idx [B, H, nb, kmax], cnt [B, H, nb] of int32, kmax < nb."""
    assert kmax < nb
    g = torch.Generator().manual_seed(seed)
    pick = torch.rand(B, H, nb, nb, generator=g).argsort(-1)[..., :kmax]
    cnt = torch.full((B, H, nb), kmax)
    if kind != "full":  # every length, many of them 0 or 1
        cnt = torch.randint(0, kmax + 1, (B, H, nb), generator=g)
        cnt[..., ::5] = 0
        cnt[..., 1::5] = 1
    live = torch.arange(kmax) < cnt[..., None]
    idx = torch.where(live, pick, torch.full_like(pick, nb)).sort(-1).values
    idx = torch.where(live, idx, torch.full_like(idx, -1)).int()
    if kind == "invalid":  # entries that name no block, first and last ones among them
        r = torch.rand(B, H, nb, kmax, generator=g)
        idx[live & (r < 0.3)] = -1
        idx[live & (r > 0.9)] = nb + 2
    return idx, cnt.int()


def valid_lists(idx, cnt, nb):
    """The same lists of one head without the entries that name no block (numpy)."""
    out = np.full(idx.shape, -1, np.int32)
    n = np.zeros(len(cnt), np.int32)
    for i in range(len(cnt)):
        row = idx[i, :cnt[i]]
        row = row[(row >= 0) & (row < nb)]
        out[i, :len(row)], n[i] = row, len(row)
    return out, n


def tensors(B, H, N, token_major, seed, qk_scale, growing):
    g = torch.Generator(device=DEV).manual_seed(seed)
    x = [torch.randn(B, H, N, 128, generator=g, device=DEV) for _ in range(3)]
    x[0] *= qk_scale
    x[1] *= qk_scale
    if growing:  # later keys score higher: the reference maximum keeps rising
        x[1] *= torch.linspace(0.2, 6, N, device=DEV)[:, None]
    out = []
    for t in x:
        d = torch.empty(B, N, H, 128, dtype=torch.bfloat16, device=DEV).permute(0, 2, 1, 3) \
            if token_major else torch.empty(B, H, N, 128, dtype=torch.bfloat16, device=DEV)
        out.append(d.copy_(t))
    return out


# B * H * ceil(N / 64) = 6144 tiles in each; N of 1000 and 1023: last tile of
# 40 and 63 rows, 993: of 33 and 449 of 1, whose second half tile is past the
# end; block 128: N mod 128 = 104, 33 and 1
CASES = [
    # B, H, N, block, lists, token-major, causal, q and k scale, growing keys
    (2, 192, 1000, 64, "full", False, None, 1.0, False),
    (2, 192, 1000, 64, "ragged", True, None, 2.0, False),
    (1, 384, 1023, 64, "invalid", True, None, 1.0, False),
    (2, 192, 993, 64, "ragged", False, None, 1.0, True),
    (2, 384, 449, 64, "invalid", False, None, 2.0, True),
    (2, 192, 1000, 128, "ragged", True, None, 1.0, True),
    (1, 384, 993, 128, "invalid", False, None, 2.0, False),
    (4, 192, 449, 128, "full", True, None, 1.0, False),
    (2, 192, 1000, 64, "full", True, (100, 0), 1.0, False),
    (2, 192, 1000, 64, "ragged", False, (100, 1), 2.0, False),
    (2, 192, 1000, 128, "ragged", True, (333, 2), 1.0, True),
    (2, 192, 1000, 64, "full", False, (17, 3), 1.0, False),
    (1, 384, 993, 128, "invalid", True, (64, 1), 1.0, False),
]


@pytest.mark.parametrize("B,H,N,block,kind,token_major,causal,qk_scale,growing", CASES)
def test_one_wave_kernel_edges(B, H, N, block, kind, token_major, causal, qk_scale, growing):
    seed = 31 * N + block + len(kind)
    nb = O.block_count(N, block)
    kmax, tiles = max(2, nb - 2), -(-N // 64)
    assert one_wave(B * H * tiles, kmax, nb, block) and not one_wave(tiles, kmax, nb, block)
    q, k, v = tensors(B, H, N, token_major, seed, qk_scale, growing)
    idx, cnt = make_lists(kind, B, H, nb, kmax, seed)
    di, dc = idx.to(DEV), cnt.to(DEV)
    order = sa.sparse_attn_schedule(dc, N, idx.shape[-1], block=block)
    kw = dict(block=block, causal=causal)
    o, lse = sa.sparse_attn_fwd(q, k, v, di, dc, order=order, o=torch.full_like(q, float("nan")),
                                **kw)
    bits = lambda t: t.contiguous().view(torch.int16)
    # raster order and no LSE
    o2, none = sa.sparse_attn_fwd(q, k, v, di, dc, with_lse=False, **kw)
    assert none is None and torch.equal(bits(o2), bits(o))
    for b, h in ((0, 0), (B - 1, H - 1), (0, H // 2)):
        alone = [t[b:b + 1, h:h + 1] for t in (q, k, v)]
        o1, l1 = sa.sparse_attn_fwd(*alone, di[b:b + 1, h:h + 1].contiguous(),
                                    dc[b:b + 1, h:h + 1].contiguous(), **kw)
        assert torch.equal(bits(o1), bits(o[b:b + 1, h:h + 1])), (b, h)
        assert torch.equal(l1, lse[b:b + 1, h:h + 1]), (b, h)
        ri, rc = valid_lists(idx[b, h].numpy(), cnt[b, h].numpy(), nb)
        x = [widen(t[0, 0].cpu()) for t in alone]
        if causal is None:
            ro, rl = O.sparse_attention(*x, ri, rc, block, TAU)[:2]
        else:
            ro, rl = O.sparse_attention_causal(*x, ri, rc, block, TAU, *causal)
        check_out(o[b, h].cpu(), None, ro, rl, what=f"b{b} h{h}")
        l = lse[b, h].cpu().double().numpy()
        live = np.isfinite(rl)
        assert np.array_equal(np.isneginf(l), ~live)
        assert np.abs(l[live] - rl[live]).max(initial=0) <= LSE_ABS


@pytest.mark.parametrize("qk_scale", [1.0, 2.0])
def test_rows_of_equal_values_come_back_exactly(qk_scale):
    """The row sum is taken over the probabilities as the product with V reads
    them (rounded to bf16), so their roundings cancel: V = 1 gives O = 1, to
    the fp32 sums' 1e-6, which is 1 in bf16.  Sums of the unrounded ones would
    leave a relative error of up to 2^-9."""
    B, H, N = 2, 192, 1000
    q, k, v = tensors(B, H, N, False, 5, qk_scale, False)
    v.fill_(1.0)
    idx, cnt = make_lists("full", B, H, 16, 13, 6)
    idx, cnt = idx.to(DEV), cnt.to(DEV)
    assert one_wave(B * H * 16, 13, 16)
    o, _ = sa.sparse_attn_fwd(q, k, v, idx, cnt)
    assert torch.equal(o, torch.ones_like(o))
    o, _ = sa.sparse_attn_fwd(q[:, :2], k[:, :2], v[:, :2], idx[:, :2].contiguous(),
                              cnt[:, :2].contiguous())
    assert torch.equal(o, torch.ones_like(o))


def _us(f, reps=10):
    f()
    torch.cuda.synchronize()
    best = float("inf")
    for _ in range(3):
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        a.record()
        for _ in range(reps):
            f()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) * 1e3 / reps)
    return best


def test_one_long_list_does_not_hold_up_the_launch():
    """A whole-head budget may keep one row whole.  The other 1022 tiles' work
    (about 105 us) runs beside such a list, so the call takes about the time
    of one long list alone on the four-wave kernel: 1.05 times it measured, and
    2.2 with one wave per tile."""
    H, N, keep = 2, 32768, 36
    nb = N // 64
    g = torch.Generator(device=DEV).manual_seed(9)
    q, k, v = (torch.randn(1, H, N, 128, generator=g, device=DEV).bfloat16() for _ in range(3))
    cnt = torch.full((1, H, nb), keep)
    cnt[..., 0] = nb
    first = (torch.arange(nb) - keep // 2).clamp(0, nb - keep)
    j = torch.arange(nb)
    idx = torch.where(j < keep, first[:, None] + j, -1)
    idx[0] = j
    idx = idx.int().expand(1, H, nb, nb).contiguous().to(DEV)
    cnt = cnt.int().to(DEV)
    order = sa.sparse_attn_schedule(cnt, N, nb)
    assert not one_wave(H * nb, nb, nb) and one_wave(H * nb, nb - 1, nb)
    both = _us(lambda: sa.sparse_attn_fwd(q, k, v, idx, cnt, order=order))
    only = cnt[:, :1].clone()  # one head: 512 tiles
    only[..., 1:] = 0
    head = [t[:, :1].contiguous() for t in (q, k, v, idx)]
    alone = _us(lambda: sa.sparse_attn_fwd(*head, only))
    print(f"  {both:.0f} us, the long list alone {alone:.0f}")
    assert both < 1.5 * alone, (both, alone)
