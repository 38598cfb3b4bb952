"""The dispatch rules between kernels of one call, on both sides of each line: the chunk counts and rank forms of the
resident anchor kernels, the item of a batch of one (kernel arguments) against the same item in a batch of two (device
scratch), and rotary keys and values in one launch or two.

Anchors: bf16 rows and coefficients are exact operands and the basis carries 16 bits, so distances are within 1e-4 of
fp64 (2^-17 of a reconstruction of RMS about 1, averaged), weights (softmax of -d at temperature 1) within 1e-3, and the
corrected rows within the bf16 bar of 1e-2 of the slice's largest value."""
import math

import pytest
import torch

from paper_2609_34060_amd import kvc

pytestmark = pytest.mark.gpu


def _pools(L, H, d, bs, blocks, dtype, seed):
    g = torch.Generator().manual_seed(seed)
    return torch.randn(L, 2, blocks, bs, H, d, generator=g).to(dtype), torch.randperm(blocks, generator=g), g


@pytest.mark.parametrize("d,ranks", [
    (128, (32,)), (128, (32, 16, 8, 32)), (128, (8,) * 5), (128, (32,) * 7), (128, (24,) * 8), (64, (32,) * 10),
    (128, (64, 32)), (128, (40, 96, 8)), (128, (64,) * 5), (128, (5, 32, 17)), (64, (33, 64, 1)), (128, (12,) * 9),
    (128, (24, 8)), (64, (64,)), (128, (3,)), (64, (7, 2, 20)), (128, (20,) * 10)])
def test_resident_anchor_chunk_counts(d, ranks):
    _check_resident(d, ranks, 1201, 1187)


# Waves with no tile, one tile and two tiles of 16 tokens (eight waves take a segment's tiles in turn).
@pytest.mark.parametrize("d,ranks,T,Ts", [
    (128, (28,) * 8, 130, 130), (64, (10, 39), 7, 5), (128, (12,), 113, 96), (128, (32,) * 10, 130, 120), (64, (8,), 16, 1)])
def test_resident_anchor_short_segments(d, ranks, T, Ts):
    _check_resident(d, ranks, T, Ts)


def _check_resident(d, ranks, T, Ts):
    L, H, bs = 1, 2, 16
    need = -(-(T + 5) // bs)
    pool, ids, g = _pools(L, H, d, bs, 2 * need, torch.bfloat16, sum(ranks) + d)
    tab = (ids[:need], ids[need:])
    off, V = (3, 5), len(ranks)
    rows = [(tab[i][(torch.arange(T) + off[i]) // bs], (torch.arange(T) + off[i]) % bs) for i in range(2)]
    dev = pool.cuda()
    cache = kvc.Cache([dev[l, 0] for l in range(L)], [dev[l, 1] for l in range(L)])

    def states():
        return [kvc.State((torch.randn(L, 2, H, Ts, r, generator=g)).to(torch.bfloat16).cuda(),
                          (torch.randn(L, 2, H, r, d, generator=g) / math.sqrt(r)).cuda()) for r in ranks]

    bases, deltas = states(), states()
    empty = kvc.State(torch.zeros(L, 2, H, 0, 0, dtype=torch.bfloat16).cuda(), torch.zeros(L, 2, H, 0, d).cuda())
    t = [x.to(torch.int32).view(1, -1).cuda() for x in tab]
    batch = kvc.Batch([T], [off[0]], [off[1]], [empty], t[0], t[1])
    an = kvc.Anchors(bases, Ts, L)
    dist = kvc.kvc_gate_distances(cache, batch, an, Ts)
    kvc.kvc_anchor_weights(cache, batch, an)
    kvc.kvc_apply_anchored(cache, batch, an.with_states(deltas))
    got = dev.cpu()

    def recon(s, l, kv):
        return torch.matmul(s.coef[l, kv].cpu().double(), s.basis[l, kv].cpu().double())  # [H, Ts, d]

    square = torch.zeros(V, dtype=torch.float64)
    for l in range(L):
        for kv in range(2):
            src = pool[l, kv][rows[0][0], rows[0][1]].double()  # [T, H, d]
            offs = [src[:Ts].transpose(0, 1) - recon(s, l, kv) for s in bases]
            dv = torch.stack([o.abs().mean(dim=(0, 2)) for o in offs], dim=-1)
            w = torch.softmax(-dv, dim=-1)
            assert (an.weights[l, kv].cpu().double() - w).abs().max() <= 1e-3
            if kv == 1:
                square += torch.stack([o.square().sum() for o in offs])
            want = src.clone()
            for v, s in enumerate(deltas):
                want[:Ts] += w[:, v, None, None] * recon(s, l, kv).transpose(0, 1)
            have = got[l, kv][rows[1][0], rows[1][1]]
            assert (have.double() - want).abs().max() <= 1e-2 * want.abs().max()
            assert torch.equal(have[Ts:], pool[l, kv][rows[0][0], rows[0][1]][Ts:])
    assert (dist.cpu().double() - square.sqrt()).abs().max() <= 1e-4 * square.sqrt().max()


@pytest.mark.parametrize("style,bs,d,T,Ts", [
    (0, 16, 128, 1100, 1000), (0, 1, 64, 600, 590), (1, 16, 128, 2101, 1030), (2, 4, 64, 1500, 1490), (2, 16, 128, 9, 9)])
def test_one_anchor_equals_the_state_applied(style, bs, d, T, Ts):
    """A single anchor has weight 1, so its apply (workgroups of their own lengths, with and without rotary keys; block
    tables in registers and, for blocks of 1 and 4 tokens, in memory) is the state's: one bf16 rounding of the value, and
    fp32 sums in another order near zero."""
    L, H, r = 2, 2, 24
    need = -(-(T + 5) // bs)
    pool, ids, g = _pools(L, H, d, bs, 2 * need, torch.bfloat16, T)
    inv = [1e4 ** (-2.0 * i / d) for i in range(d // 2)] if style else None
    st = kvc.State(torch.randn(L, 2, H, Ts, r, generator=g).to(torch.bfloat16).cuda(),
                   (torch.randn(L, 2, H, r, d, generator=g) / math.sqrt(r)).cuda())
    empty = kvc.State(torch.zeros(L, 2, H, 0, 0, dtype=torch.bfloat16).cuda(), torch.zeros(L, 2, H, 0, d).cuda())
    tabs = [ids[i * need:(i + 1) * need].to(torch.int32).view(1, -1).cuda() for i in range(2)]
    pos = dict(src_positions=[7], dst_positions=[300]) if style else {}
    found = []
    for item in (empty, st):
        dev = pool.cuda()
        cache = kvc.Cache([dev[l, 0] for l in range(L)], [dev[l, 1] for l in range(L)], rope_style=style,
                          rope_inv_freq=inv)
        batch = kvc.Batch([T], [5], [2], [item], *tabs, **pos)
        if item is empty:
            an = kvc.Anchors([st], Ts, L)
            kvc.kvc_anchor_weights(cache, batch, an)
            assert bool((an.weights == 1.0).all())
            kvc.kvc_apply_anchored(cache, batch, an)
        else:
            kvc.kvc_apply(cache, batch)
        found.append(dev.cpu().float())
    a, b = found
    assert ((a - b).abs() <= b.abs() * 2.0 ** -7 + 2.0 ** -14).all()
    assert not torch.equal(b, pool.float())


@pytest.mark.parametrize("dtype,d,style", [(torch.bfloat16, 128, 0), (torch.bfloat16, 128, 1), (torch.bfloat16, 64, 2),
                                           (torch.float32, 128, 0), (torch.float32, 64, 1)])
def test_one_item_equals_the_same_item_in_a_batch(dtype, d, style):
    """Items that differ in every field: rows and states of each alone (its item in the kernel arguments) against the
    batch of both (items in the device scratch).  Applies agree bit for bit, and so does the first item's fit.  The second
    item's units have other numbers in the batch and with them other start vectors of the inverse iteration: the same
    singular values, basis rows within a few fp32 roundings, coefficients within those or one rounding to storage."""
    L, H, bs, n = 2, 3, 16, 2
    T, r, off, pos = (333, 517), (12, 40), ((7, 2), (0, 21)), ((4, 90), (31, 8))
    need = -(-(max(T) + 21) // bs)
    pool, ids, g = _pools(L, H, d, bs, 2 * n * need, dtype, d + style)
    inv = [1e4 ** (-2.0 * i / d) for i in range(d // 2)] if style else None
    tabs = ids.to(torch.int32).view(2, n, need).cuda()
    states = [kvc.State(torch.randn(L, 2, H, T[i] - 9 * i, r[i], generator=g).to(dtype).cuda(),
                        torch.randn(L, 2, H, r[i], d, generator=g).cuda()) for i in range(n)]

    def run(items):
        dev = pool.cuda()
        cache = kvc.Cache([dev[l, 0] for l in range(L)], [dev[l, 1] for l in range(L)], rope_style=style,
                          rope_inv_freq=inv)
        out = [kvc.State.empty(L, H, d, T[i], r[i], dtype, "cuda") for i in items]

        def batch(st):
            p = dict(src_positions=[pos[i][0] for i in items], dst_positions=[pos[i][1] for i in items]) if style else {}
            return kvc.Batch([T[i] for i in items], [off[i][0] for i in items], [off[i][1] for i in items], st,
                             tabs[0][items], tabs[1][items], **p)

        kvc.kvc_fit_state(cache, batch(out))
        kvc.kvc_apply(cache, batch([states[i] for i in items]))
        rows = [dev[:, :, tabs[1][i].long()].cpu() for i in items]
        return rows, [(o.coef.cpu().double(), o.basis.cpu().double(), o.sigma.cpu()) for o in out]

    both = run([0, 1])
    for i in range(n):
        alone = run([i])
        assert torch.equal(alone[0][0], both[0][i])
        a, b = alone[1][0], both[1][i]
        assert torch.equal(a[2], b[2])
        if i == 0:
            assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
        else:
            assert (a[1] - b[1]).abs().max() <= 1e-5
            rounding = 2.0 ** -8 if dtype == torch.bfloat16 else 1e-5
            assert (a[0] - b[0]).abs().max() <= rounding * a[0].abs().max()


@pytest.mark.parametrize("lengths,L", [
    ((100,), 47), ((100,), 48), ((520,), 24), ((520,), 25), ((900,), 47), ((900,), 48), ((1030,), 87), ((1030,), 88),
    ((1540,), 23), ((1540,), 24), ((2048,), 25), ((2300,), 37), ((2300,), 38), ((700, 130, 512) * 4, 2),
    ((700, 130, 512) * 4 + (1,), 2), ((1700, 400) * 4, 2), ((1700, 400) * 5, 2), ((1300, 1025, 3) * 5, 1)])
def test_rotary_apply_in_one_launch_or_two(lengths, L):
    """Sizes on both sides of the lines between a joint launch of keys and values and separate ones: a call over all
    layers equals calls of one layer each (whose few workgroups take the joint launch), bit for bit."""
    H, d, r, bs, n = 8, 128, 20, 16, len(lengths)
    need = -(-(max(lengths) + 7) // bs)
    g = torch.Generator(device="cuda").manual_seed(L + n)
    pool = torch.randn(L, 2, 2 * n * need, bs, H, d, generator=g, device="cuda").to(torch.bfloat16)
    ids = torch.randperm(2 * n * need, generator=g, device="cuda").to(torch.int32).view(2, n, need)
    st = []
    for t in lengths:
        ts = max(1, t - 5)
        st.append(kvc.State(torch.randn(L, 2, H, ts, r, generator=g, device="cuda").to(torch.bfloat16),
                            torch.randn(L, 2, H, r, d, generator=g, device="cuda")))
    batch = kvc.Batch(lengths, [7] * n, [3] * n, st, ids[0], ids[1], src_positions=[4 + i for i in range(n)],
                      dst_positions=[90] * n)
    inv = [1e4 ** (-2.0 * i / d) for i in range(d // 2)]
    got = []
    for step in (L, 1):
        dev = pool.clone()
        cache = kvc.Cache([dev[l, 0] for l in range(L)], [dev[l, 1] for l in range(L)], rope_style=kvc.KVC_ROPE_HALF,
                          rope_inv_freq=inv)
        for l in range(0, L, step):
            kvc.kvc_apply(cache, batch, l, l + step)
        got.append(dev)
    assert torch.equal(got[0], got[1])
    assert not torch.equal(got[0], pool)
