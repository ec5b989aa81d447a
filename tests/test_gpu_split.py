"""GPU parity of the split-key cache kernels (ism_split.hip, and the forward
kernel over the same plan) where the plan and the tiles can go wrong: column
counts (new rows x query heads per KV head) around one 32-column block,
histories at the edges of the 32-key tiles, more dialogues than lanes of the
planning wave, dialogues without new rows, ragged lengths that are cut into one
to many chunks, decode workspaces from the smallest to more than is used,
prefill workspaces from none to full, and out-of-contract lengths. Against the fp64 oracle, with outputs filled
with NaN; paged equal to dense bit for bit, and the caches after the append
equal to the inputs.
"""

import numpy as np
import pytest

import oracle
from paper_2408_00539_amd import workloads as W
from tests._gpu import announce, compare, dev_bf16, f64, host_f64, torch_cuda

pytestmark = pytest.mark.gpu


def _bits(rng, *shape):
    return W.to_bf16_bits(rng.standard_normal(shape, dtype=np.float32))


def _hist(rng, batch, longest):
    edges = [min(x, longest) for x in (0, 1, 31, 32, 33, 63, 64, 127, 128, 129, longest)]
    more = rng.integers(0, longest + 1, size=max(0, batch - len(edges)))
    return np.concatenate([edges, more])[:batch].astype(np.int32)


@pytest.mark.parametrize("batch,longest,hq,hkv,d,new,is_query", [
    (11, 2100, 8, 2, 128, 8, False),    # 32 columns, many chunks
    (11, 2100, 3, 1, 64, 10, False),    # 30 columns, group of 3
    (11, 700, 8, 2, 128, 9, True),      # 36 columns: row-tiled
    (5, 130, 1, 1, 64, 32, False),      # no grouping
    (70, 300, 4, 1, 128, 4, False),     # more dialogues than lanes
    (130, 90, 2, 2, 64, 3, True),
    (260, 70, 16, 8, 64, 3, False),     # 2080 workgroups: whole dialogues, no plan
    # more chunks wanted than the chip holds, so that their length is searched:
    # one wave of dialogues, two, three, more than the registers hold
    (40, 2100, 8, 8, 64, 8, False),
    (70, 1500, 8, 8, 64, 4, True),
    (130, 700, 16, 8, 64, 3, False),
    (300, 500, 2, 1, 64, 3, False),
    # the row-tiled kernel over split key ranges: chunks that some or all rows
    # of a workgroup end before, several column groups, heads of a group of 3
    (4, 2100, 4, 1, 128, 150, False),
    (5, 1300, 2, 2, 64, 200, False),
    (11, 900, 16, 1, 64, 40, True),
    (3, 5000, 3, 1, 128, 33, False),
    (8, 9000, 4, 4, 64, 100, False),
    (11, 1100, 16, 1, 64, 40, True),
    # the row-tiled kernel with a group's heads in two and four sets
    (4, 700, 32, 2, 64, 230, False),
    (2, 300, 192, 3, 64, 300, True),
    # one new row whose heads alone fill more than one 32-column block
    (5, 4000, 40, 1, 64, 1, True),
    (4, 8000, 64, 1, 128, 1, False),
    (3, 4100, 160, 1, 64, 1, False),
    (11, 1100, 256, 1, 128, 1, True),
    (5, 1300, 512, 2, 128, 1, False),
])
def test_ragged_chunks(batch, longest, hq, hkv, d, new, is_query):
    torch = torch_cuda()
    from paper_2408_00539_amd import ops
    rng = np.random.default_rng(batch * 7 + longest + hq + d + new)
    hist = _hist(rng, batch, longest)
    lens = rng.integers(0, new + 1, size=batch)  # some dialogues get no row
    lens[:2] = new
    cap, ps = -(-(longest + new) // 64) * 64, 64
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    kc, vc = _bits(rng, batch, hkv, cap, d), _bits(rng, batch, hkv, cap, d)
    q, k, v = (_bits(rng, cu[-1], n, d) for n in (hq, hkv, hkv))
    Kc, Vc = dev_bf16(kc), dev_bf16(vc)
    mp = cap // ps
    order = rng.permutation(batch * mp + 3)[:batch * mp].reshape(batch, mp).astype(np.int32)
    Kp = torch.zeros((batch * mp + 3, hkv, ps, d), dtype=torch.bfloat16, device="cuda")
    Vp = torch.zeros_like(Kp)
    tab = torch.from_numpy(order).cuda()
    for pool, cache in ((Kp, Kc), (Vp, Vc)):
        pool[tab.long().reshape(-1)] = cache.view(batch, hkv, mp, ps, d).transpose(1, 2).reshape(
            batch * mp, hkv, ps, d)
    dev = dev_bf16(q), dev_bf16(k), dev_bf16(v)
    tl, tc = torch.from_numpy(hist).cuda(), torch.from_numpy(cu).cuda()
    o = torch.full((int(cu[-1]), hq, d), float("nan"), dtype=torch.bfloat16, device="cuda")
    lse = torch.full((hq, int(cu[-1])), float("nan"), device="cuda")
    announce("split chunks", batch, longest, hq, hkv, d, new, is_query)
    ops.prefill_cached_segment(*dev, Kc, Vc, tl, tc, new, is_query, out=(o, lse))
    op, lp = ops.prefill_paged(*dev, Kp, Vp, tab, tl, tc, new, is_query)
    torch.cuda.synchronize()
    assert torch.equal(o.view(torch.int16), op.view(torch.int16)) and torch.equal(lse, lp)
    ro, rl = np.empty((cu[-1], hq, d)), np.empty((hq, cu[-1]))
    for b in range(batch):
        r, C, L = slice(cu[b], cu[b + 1]), int(hist[b]), int(lens[b])
        if not L:
            continue
        ro[r], rl[:, r], _, _ = oracle.prefill_cached(
            f64(kc[b, :, :C]).transpose(1, 0, 2), f64(vc[b, :, :C]).transpose(1, 0, 2), f64(q[r]),
            f64(k[r]), f64(v[r]), 1 / np.sqrt(d), new_is_query=is_query)
        kc[b, :, C:C + L] = k[r].transpose(1, 0, 2)
        vc[b, :, C:C + L] = v[r].transpose(1, 0, 2)
    compare("O split", host_f64(o), ro)
    compare("LSE split", host_f64(lse), rl)
    for cache, pool, want in ((Kc, Kp, kc), (Vc, Vp, vc)):
        np.testing.assert_array_equal(cache.view(torch.int16).cpu().numpy().view(np.uint16), want)
        back = pool[tab.long().reshape(-1)].view(batch, mp, hkv, ps, d).transpose(1, 2).reshape(
            batch, hkv, cap, d)
        assert torch.equal(back.view(torch.int16), cache.view(torch.int16))


@pytest.mark.parametrize("ps", [64, 128, 192, 448])
@pytest.mark.parametrize("longest,hq,hkv,d,new,is_query", [
    (8200, 64, 32, 64, 150, False),   # row tiles, transfers spread over the step
    (8200, 48, 24, 128, 70, True),    # one and two column tiles
    (9000, 4, 4, 128, 100, False),    # the same over split key ranges
    (700, 64, 32, 64, 150, True),     # a short cache: transfers at once
    (3000, 8, 2, 128, 8, False),      # the split-key kernel
])
def test_page_sizes(ps, longest, hq, hkv, d, new, is_query):
    """Pages of one tile and of several, ragged histories that end at their
    edges: the dense cache's bits."""
    torch = torch_cuda()
    from paper_2408_00539_amd import ops
    rng = np.random.default_rng(ps + longest + d)
    hist = np.array([longest, 5 * ps - new, 2 * ps - 1, 64 * 3, 0], np.int32)
    lens = np.array([new, new, max(1, new // 3), 1, new], np.int32)
    B, mp = len(hist), -(-(longest + new) // ps)
    hist = np.clip(hist, 0, mp * ps - lens)
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    gen = torch.Generator(device="cuda").manual_seed(int(rng.integers(1 << 30)))
    rand = lambda *s: torch.randn(s, generator=gen, device="cuda").bfloat16()
    Kc, Vc = rand(B, hkv, mp * ps, d), rand(B, hkv, mp * ps, d)
    tab = torch.from_numpy(rng.permutation(B * mp + 3)[:B * mp].reshape(B, mp).astype(np.int32)).cuda()
    pools = []
    for cache in (Kc, Vc):
        pools.append(rand(B * mp + 3, hkv, ps, d))
        pools[-1][tab.long().reshape(-1)] = cache.view(B, hkv, mp, ps, d).transpose(1, 2).reshape(
            B * mp, hkv, ps, d)
    q, k, v = (rand(int(cu[-1]), n, d) for n in (hq, hkv, hkv))
    tl, tc = torch.from_numpy(hist).cuda(), torch.from_numpy(cu).cuda()
    announce("page sizes", ps, longest, hq, hkv, d, new, is_query)
    o, lse = ops.prefill_cached_segment(q, k, v, Kc, Vc, tl, tc, new, is_query)
    op, lp = ops.prefill_paged(q, k, v, *pools, tab, tl, tc, new, is_query)
    torch.cuda.synchronize()
    assert torch.equal(o.view(torch.int16), op.view(torch.int16)) and torch.equal(lse, lp)
    assert torch.isfinite(lse).all()
    for cache, pool in zip((Kc, Vc), pools):
        back = pool[tab.long().reshape(-1)].view(B, mp, hkv, ps, d).transpose(1, 2).reshape(
            B, hkv, mp * ps, d)
        assert torch.equal(back.view(torch.int16), cache.view(torch.int16))


def _least_decode_workspace(B, max_len, hq, hkv, d, splits):
    """The smallest workspace a matrix-core decode step accepts: the partials
    of one chunk per 256 keys, at most 64 and at most 768 head sets, or of the
    asked-for chunks."""
    g = hq // hkv
    sets = hq // max(x for x in range(1, min(g, 32) + 1) if g % x == 0)
    s = splits or max(1, min(-(-768 // (B * sets)), -(-max_len // 256), 64))
    up = lambda n: -(-n // 256) * 256
    return up(B * hq * s * d * 4) + up(B * hq * s * 8)


@pytest.mark.parametrize("hq,hkv,d,cap,splits", [
    (8, 2, 128, 3000, 0),    # 4 columns
    (40, 1, 64, 3000, 0),    # 40: two column groups
    (33, 1, 64, 256, 0),     # the smallest holds one chunk per dialogue
    (8, 2, 128, 3000, 7),    # asked-for chunks, and fewer in a smaller one
    (33, 1, 64, 900, 3),     # one of three
])
def test_decode_workspaces(hq, hkv, d, cap, splits):
    """The same step in workspaces from the smallest that is accepted (fewer
    chunks, down to one per dialogue) to more than it uses, and 256 bytes less
    than the smallest (refused); one dialogue's position lies outside the cache
    (NaN, nothing appended)."""
    torch = torch_cuda()
    from paper_2408_00539_amd import ops
    rng = np.random.default_rng(hq + d + cap + splits)
    pos = np.array([0, 1, 31, 32, cap - 1, cap, cap // 2, cap // 4, 64], np.int32)
    B = len(pos)
    kc, vc = _bits(rng, B, hkv, cap, d), _bits(rng, B, hkv, cap, d)
    q, k, v = _bits(rng, B, hq, d), _bits(rng, B, hkv, d), _bits(rng, B, hkv, d)
    want = [oracle.decode_step(f64(kc[b, :, :p]).transpose(1, 0, 2),
                               f64(vc[b, :, :p]).transpose(1, 0, 2), f64(q[b]), f64(k[b]),
                               f64(v[b]), 1 / np.sqrt(d))[:2] if p < cap else None
            for b, p in enumerate(pos)]
    full = ops.workspace_size(ops.ISM_OP_DECODE, B, 0, cap, hq, hkv, d, splits)
    least = _least_decode_workspace(B, cap, hq, hkv, d, splits)
    assert least < full

    def step(nbytes):
        Kc, Vc = dev_bf16(kc), dev_bf16(vc)
        ws = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        announce("decode workspace", hq, hkv, d, cap, splits, nbytes)
        return (Kc, *ops.decode(dev_bf16(q), dev_bf16(k), dev_bf16(v), Kc, Vc,
                                torch.from_numpy(pos).cuda(), workspace=ws, num_splits=splits))

    with pytest.raises(ops.IsmError, match="ISM_ERR_WORKSPACE"):
        step(least - 256)
    for nbytes in (least, least + 4096, (least + full) // 512 * 256, full - 256, full, full + 4096):
        Kc, o, lse = step(nbytes)
        o, lse = host_f64(o), host_f64(lse)
        got = Kc.view(torch.int16).cpu().numpy().view(np.uint16)
        for b, p in enumerate(pos):
            if p >= cap:
                assert np.isnan(o[b]).all() and np.isnan(lse[:, b]).all()
                np.testing.assert_array_equal(got[b], kc[b])
                continue
            compare(f"O ws {nbytes} b{b}", o[b], want[b][0])
            compare(f"LSE ws {nbytes} b{b}", lse[:, b], want[b][1])
            np.testing.assert_array_equal(got[b, :, p], k[b])


@pytest.mark.parametrize("longest,hq,hkv,d,new,is_query", [
    (2100, 8, 2, 128, 8, False),      # 32 columns: split, or row-tiled with an append launch
    (2100, 4, 1, 128, 150, True),     # row-tiled: split, or not
    (4000, 64, 1, 64, 1, False),
])
def test_prefill_workspaces(longest, hq, hkv, d, new, is_query):
    """A prefill that would split its keys, given no workspace, one that is too
    small or misaligned, and its own: the oracle's result and the same caches in
    each, paged equal to dense bit for bit."""
    torch = torch_cuda()
    from paper_2408_00539_amd import ops
    rng = np.random.default_rng(longest + hq + new)
    B, ps = 5, 64
    hist = np.array([longest, longest // 2, 129, 64, 0], np.int32)
    lens = np.array([new, max(1, new // 2), 1, new, new], np.int32)
    cap = -(-(longest + new) // ps) * ps
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    Tn, mp = int(cu[-1]), cap // ps
    kc, vc = _bits(rng, B, hkv, cap, d), _bits(rng, B, hkv, cap, d)
    q, k, v = (_bits(rng, Tn, n, d) for n in (hq, hkv, hkv))
    need = ops.prefill_workspace_size(B, Tn, new, hq, hkv, d, cap)
    assert need > 0
    ro, rl = np.empty((Tn, hq, d)), np.empty((hq, Tn))
    want_k = kc.copy()
    for b in range(B):
        r, C, L = slice(cu[b], cu[b + 1]), int(hist[b]), int(lens[b])
        ro[r], rl[:, r], _, _ = oracle.prefill_cached(
            f64(kc[b, :, :C]).transpose(1, 0, 2), f64(vc[b, :, :C]).transpose(1, 0, 2), f64(q[r]),
            f64(k[r]), f64(v[r]), 1 / np.sqrt(d), new_is_query=is_query)
        want_k[b, :, C:C + L] = k[r].transpose(1, 0, 2)
    dev = dev_bf16(q), dev_bf16(k), dev_bf16(v)
    tl, tc = torch.from_numpy(hist).cuda(), torch.from_numpy(cu).cuda()
    tab = torch.from_numpy(rng.permutation(B * mp).reshape(B, mp).astype(np.int32)).cuda()
    ws = torch.empty(need + 512, dtype=torch.uint8, device="cuda")
    ptr = lambda t: t.data_ptr()
    stream, scale = torch.cuda.current_stream().cuda_stream, 1 / np.sqrt(d)
    for off, nbytes in ((None, 0), (0, need - 256), (128, need), (0, need)):
        got = []
        for paged in (False, True):
            Kc, Vc = dev_bf16(kc), dev_bf16(vc)
            if paged:
                pools = []
                for cache in (Kc, Vc):
                    pools.append(torch.zeros((B * mp, hkv, ps, d), dtype=cache.dtype, device="cuda"))
                    pools[-1][tab.long().reshape(-1)] = cache.view(B, hkv, mp, ps, d).transpose(
                        1, 2).reshape(B * mp, hkv, ps, d)
            o = torch.full((Tn, hq, d), float("nan"), dtype=torch.bfloat16, device="cuda")
            lse = torch.full((hq, Tn), float("nan"), device="cuda")
            tail = (ptr(o), ptr(lse), hq, hkv, d, scale, None if off is None else ptr(ws) + off,
                    nbytes, stream)
            announce("prefill workspace", longest, hq, hkv, d, new, is_query, off, nbytes, paged)
            head = (ptr(tc), B, Tn, new, int(is_query), *map(ptr, dev))
            if paged:
                st = ops.lib().ism_attn_prefill_paged(*head, *map(ptr, pools), B * mp, ps, ptr(tab),
                                                      mp, ptr(tl), *tail)
            else:
                st = ops.lib().ism_attn_prefill_cached_segment(*head, ptr(Kc), ptr(Vc), cap, ptr(tl),
                                                               *tail)
            assert st == 0
            torch.cuda.synchronize()
            if paged:
                Kc = pools[0][tab.long().reshape(-1)].view(B, mp, hkv, ps, d).transpose(
                    1, 2).reshape(B, hkv, cap, d)
            np.testing.assert_array_equal(Kc.view(torch.int16).cpu().numpy().view(np.uint16), want_k)
            got.append((o, lse))
        assert torch.equal(got[0][0].view(torch.int16), got[1][0].view(torch.int16))
        assert torch.equal(got[0][1], got[1][1])
        compare(f"O ws {off} {nbytes}", host_f64(got[0][0]), ro)
        compare(f"LSE ws {off} {nbytes}", host_f64(got[0][1]), rl)
