"""Attention rows that leave the reference-0 form of the softmax, or never have it: one,
two and four key groups, every block grid, against float64. Each row follows a profile of
its largest logit per 64-key chunk, so that chunks leave the range upwards and downwards
at odd and even places of a group's list, in one group and not in another, and groups of
comparable mass end with different references. The float64 logits are asked for each of
these before anything is compared."""
import numpy as np
import pytest

from launch_rules import attn_groups

pytestmark = pytest.mark.gpu

SCALE_LOG2 = np.float32(0.125) * np.float32(1.4426950408889634)
LIMIT, TINY, BAND = 50.0, -100.0, 24.0  # base-2 sums a chunk and a row may have, logits of the first chunk

# Largest base-2 logit of a row in chunk c of its list (one key; the others are 12 lower).
PROFILES = [
    lambda c: 10.0,                                                  # stays in range
    lambda c: {3: 80.0, 4: 78.0}.get(c, 10.0),                       # leaves at an odd and at an even chunk
    lambda c: {6: 45.0, 8: 54.0, 9: 53.0, 13: 140.0}.get(c, 0.0),    # ... later, and twice
    lambda c: -160.0 if c % 2 else 0.0,                              # every other chunk without mass
    lambda c: {2: -149.0, 9: 60.0}.get(c, -150.0),                   # starts far below, jumps up
    lambda c: {10: 190.0, 11: 189.0}.get(c, 100.0),                  # starts far above, rises out of range
    lambda c: -200.0 + 3.0 * c,
    lambda c: 300.0 if c == 0 else -300.0,
]

#        H    N             bq   bk   groups
CASES = [(256, 26 * 64 - 5, 64, 64, 1), (256, 26 * 64 - 5, 64, 128, 1), (256, 26 * 64 - 5, 128, 64, 1),
         (256, 26 * 64 - 5, 128, 128, 1), (1, 26 * 64, 64, 64, 2), (2, 27 * 64 - 63, 64, 128, 2),
         (1, 27 * 64 - 40, 128, 64, 2), (2, 26 * 64 - 1, 128, 128, 2), (1, 70 * 64 - 5, 64, 64, 4),
         (2, 67 * 64 + 1, 64, 128, 4), (1, 66 * 64, 128, 64, 4), (2, 71 * 64 - 64, 128, 128, 4)]


def layer(N):
    """Q, K, V (bf16 [N][64]) and each token's profile. Profile p has channel p to itself; tokens 0-255 hold
    one profile per wave of 32, 256-511 waves that mix the first four (those that start in range), the rest
    waves that mix all."""
    import torch

    gen = torch.Generator().manual_seed(N)
    q, k, v = (torch.randn(N, 64, generator=gen) * s for s in (0.3, 0.3, 1.0))
    t = torch.arange(N)
    prof = torch.where(t < 256, t // 32, torch.where(t < 512, t % 4, t % 8))
    q[:, :8] = 16.0 * torch.nn.functional.one_hot(prof, 8)
    for p, level in enumerate(PROFILES):
        lv = torch.tensor([level(c) for c in range(-(-N // 64))])[t // 64] - 12.0 * (t % 64 != 17)
        k[:, p] = lv / (16.0 * float(SCALE_LOG2))
    return q.bfloat16(), k.bfloat16(), v.bfloat16(), prof


def logits(q, k):
    """Base-2 logits as the kernel forms them (a wave whose first 64 lie within the band scales Q first), and
    which rows start that way."""
    import torch

    scaled = (q.float() * float(SCALE_LOG2)).bfloat16().double() @ k.double().T
    exact = (q.double() @ k.double().T) * float(SCALE_LOG2)
    inside = scaled[:, :64].max(1).values.abs() <= BAND
    inside = torch.stack([w.all() for w in inside.split(32)]).repeat_interleave(32)[:q.shape[0]]
    return torch.where(inside[:, None], scaled, exact), inside


def check_profiles(L, inside, prof, G):
    """What the cases are there for does happen: see the module's first lines."""
    import torch

    sums = torch.stack([torch.logsumexp(x * np.log(2.0), 1) / np.log(2.0) for x in L.split(64, 1)], 1)  # [row][chunk]
    left, parted = set(), False
    for w in range(8):  # the waves of one profile
        if not bool(inside[32 * w]):
            continue
        out = []
        for g in range(G):
            s = sums[32 * w:32 * w + 32, g::G]
            gone = (s > LIMIT + 1.0).any(0) | (s[:, 0] < TINY - 1.0).any() & (torch.arange(s.shape[1]) == 0)
            near = ((s > LIMIT - 1.0) & (s < LIMIT + 1.0)).any()
            assert not bool(near)
            out.append(int(gone.nonzero()[0]) if bool(gone.any()) else -1)
        left |= {x % 2 for x in out if x > 0}
        parted |= min(out) < 0 <= max(out)
    assert left == {0, 1}, "chunks that leave the range at odd and at even places"
    if G > 1:
        assert parted, "a group that leaves the range beside one that does not"
        # A new reference lies at the largest logit so far: groups that both rose, within 2^4 of each other in mass.
        top = torch.stack([sums[:, g::G].max(1).values for g in range(G)], 1).sort(1, descending=True).values
        merged = (top[:, 1] > LIMIT) & (top[:, 0] - top[:, 1] < 4.0) & (top[:, 0] - top[:, 1] > 0.5)
        assert int(merged.sum()) >= 32
    starts = L[:, :64].max(1).values
    assert bool((starts < TINY).any()) and bool((starts > LIMIT).any())


@pytest.mark.parametrize("H,N,bq,bk,G", CASES)
def test_references(H, N, bq, bk, G):
    import torch

    import paper_2609_35593_amd as ress

    n_qb, n_kb = -(-N // bq), -(-N // bk)
    assert attn_groups(H, n_qb, n_kb, bq, bk) == G
    q, k, v, prof = layer(N)
    L, inside = logits(q, k)
    check_profiles(L, inside, prof, G)
    count = torch.full((H, n_qb), n_kb, dtype=torch.int32, device="cuda")
    idx = torch.arange(n_kb, dtype=torch.int32, device="cuda").expand(H, n_qb, n_kb).contiguous()
    dev = [x.cuda().expand(H, N, 64).contiguous() for x in (q, k, v)]
    o32 = ress.ress_sparse_attn_out_f32(*dev, count, idx, bq=bq, bk=bk)
    assert bool((o32 == o32[0]).all())  # every head holds the same layer
    assert torch.equal(ress.ress_dense_attn(*dev, bq=bq, bk=bk), o32.bfloat16())
    got = o32[0].cpu().double()
    assert bool(torch.isfinite(got).all())
    w = torch.exp2(L - L.max(1, keepdim=True).values)
    w /= w.sum(1, keepdim=True)
    ref = w @ v.double()
    # A weight is rounded to bf16 (8 significant bits: off by at most 2^-8 of it) before the product and in the row's
    # sum, and its logit, up to 300 in base 2, carries float32 rounding (2^-24 of it in each of its few steps: under
    # 2^-13 in all). With weights off by a factor 1 + e, |e| <= 2^-8 + 2^-13, the output moves by at most
    # e sum_j w_j |v_j - out| / (1 - e); float32 sums add 2^-16 of sum_j w_j |v_j|.
    spread = torch.stack([(w[i:i + 1] @ (v.double() - ref[i]).abs())[0] for i in range(N)])
    bound = (2.0 ** -8 + 2.0 ** -13) * 1.01 * spread + 2.0 ** -16 * (w @ v.double().abs())
    over = ((got - ref).abs() / bound).max(1).values
    assert float(over.max()) <= 1.0, [(int(p), float(over[prof == p].max())) for p in prof.unique()]


@pytest.mark.parametrize("H,N,bq,bk", [(1, 700, 64, 64), (1, 4500, 128, 128), (256, 850, 64, 128)])
def test_first_references_round_like_zero(H, N, bq, bk):
    """Waves that start outside the band with logits of up to 49: their references are whole numbers, so the
    probabilities round to bf16 as 2^logit does, and the output is that of the weights so rounded (an eighth of the
    rounding's own effect is left for exponentials that land on the other side of a rounding boundary)."""
    import torch

    import paper_2609_35593_amd as ress

    gen = torch.Generator().manual_seed(N)
    q, k, v = (torch.randn(N, 64, generator=gen) for _ in range(3))
    q, k, v = (5.5 * q).bfloat16(), k.bfloat16(), v.bfloat16()
    q[::32] = (30.0 / float(SCALE_LOG2) / k[0].float().square().sum() * k[:1].float()).bfloat16()  # 30 in every wave
    L, inside = logits(q, k)
    assert not bool(inside.any()) and float(L.max()) < 49.0
    dev = [x.cuda().expand(H, N, 64).contiguous() for x in (q, k, v)]
    n_qb, n_kb = -(-N // bq), -(-N // bk)
    count = torch.full((H, n_qb), n_kb, dtype=torch.int32, device="cuda")
    idx = torch.arange(n_kb, dtype=torch.int32, device="cuda").expand(H, n_qb, n_kb).contiguous()
    got = ress.ress_sparse_attn_out_f32(*dev, count, idx, bq=bq, bk=bk)[0].cpu().double()
    w = torch.exp2(L)
    ref = (w / w.sum(1, keepdim=True)) @ v.double()
    w = w.float().bfloat16().double()
    rounded = (w / w.sum(1, keepdim=True)) @ v.double()
    assert float((got - rounded).norm()) <= 0.125 * float((rounded - ref).norm())
