"""The wavefronts of a decode split: the split's 64-token steps are shared by
four wavefronts whose softmax states are merged. Lengths sit on the edges of
the shares, and a sequence must come out the same alone as in a batch."""
import numpy as np
import pytest
import torch

import paper_2608_23658_amd.kvattn as K
from workloads import make_batch_from_lens
from tests.gpu_helpers import Dev, assert_parity, oracle_decode, require_gpu, say, seq_bounds

pytestmark = pytest.mark.gpu

# one step per wavefront, one more than that, uneven shares, whole splits
EDGES = [1, 64, 65, 128, 129, 192, 193, 256, 257, 320, 321, 512, 513, 960, 961, 1024, 1025,
         1088, 1089, 1280, 2047]


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def _batch(lens, hq, hkv, d, dtype, seed):
    return make_batch_from_lens(lens, [1] * len(lens), dtype=dtype, num_q_heads=hq,
                                num_kv_heads=hkv, head_dim=d, block_size=16, seed=seed)


@pytest.mark.parametrize("hq,hkv,d,dtype", [(8, 1, 128, "bf16"), (4, 4, 128, "bf16"),
                                            (16, 2, 64, "bf16"), (8, 2, 64, "f32")])
def test_share_edges(hq, hkv, d, dtype):
    b = _batch(EDGES, hq, hkv, d, dtype, seed=211)
    say("decode share edges", hq, hkv, d, dtype)
    out = Dev(b).decode()
    torch.cuda.synchronize()
    assert_parity(out, oracle_decode(b), dtype, f"share edges {hq}/{hkv}/{d}/{dtype}",
                  seq_bounds(b, decode=True))


def test_a_sequence_does_not_depend_on_its_batch():
    """Every sequence decoded on its own, with its own length as max_seq_len,
    gives the bits it gives in a batch with a far longer one."""
    b = _batch(EDGES + [9300], 8, 2, 128, "bf16", seed=212)
    dev = Dev(b)
    say("decode batch independence")
    whole = dev.decode()
    for s, L in enumerate(b.seq_lens.tolist()):
        one = K.decode(dev.q[s:s + 1], dev.kv, b.num_blocks, dev.bt[s:s + 1].contiguous(),
                       dev.sl[s:s + 1].contiguous(), num_kv_heads=2, max_seq_len=L,
                       scale=b.scale)
        assert torch.equal(one[0].view(torch.int16), whole[s].view(torch.int16)), L


def test_a_share_without_valid_blocks_contributes_nothing():
    """All blocks of one wavefront's share carry ids outside the layer; the
    result is that of the sequence without those tokens."""
    b = _batch([1024], 4, 1, 128, "bf16", seed=213)
    dev = Dev(b)
    keep = np.r_[0:16, 32:64]                      # blocks of shares 0, 2 and 3
    holes = dev.bt.clone()
    holes[0, 16:32] = b.num_blocks
    short = torch.full_like(dev.bt, -1)
    short[0, :48] = dev.bt[0, torch.from_numpy(keep).cuda()]
    say("decode share without valid blocks")
    kw = dict(num_kv_heads=1, scale=b.scale)
    got = K.decode(dev.q, dev.kv, b.num_blocks, holes, dev.sl, max_seq_len=1024, **kw)
    want = K.decode(dev.q, dev.kv, b.num_blocks, short, torch.full_like(dev.sl, 768),
                    max_seq_len=1024, **kw)
    assert torch.isfinite(got).all()
    # the two order their sums differently: P rounded to bf16 against different maxima
    d = (got.float() - want.float()).norm() / want.float().norm()
    assert d < 1e-2, float(d)


@pytest.mark.parametrize("hq,hkv,d,dtype", [(4, 1, 64, "bf16"), (2, 2, 128, "bf16"),
                                            (2, 1, 64, "f32")])
def test_combine_split_counts(hq, hkv, d, dtype):
    """1, 2, 8 (one wavefront), 9, 31, 32, 33 and 65 to 69 splits (shared by
    four wavefronts, with and without a remainder) in one batch and, for the
    lengths one wavefront merges, in a batch that has no longer ones."""
    lens = [1000, 1025, 8192, 8193, 31 * 1024, 32 * 1024, 32 * 1024 + 1, 65 * 1024 + 5,
            69 * 1024]
    for sel in (lens, lens[:3]):
        b = _batch(sel, hq, hkv, d, dtype, seed=214)
        say("decode combine", hq, hkv, d, dtype, sel)
        out = Dev(b).decode()
        torch.cuda.synchronize()
        assert_parity(out, oracle_decode(b), dtype, f"combine {hq}/{hkv}/{d}/{dtype}",
                      seq_bounds(b, decode=True))


def _least_workspace(rows, d):
    """A workspace with a partial per split of `rows` (sequence, head, split) rows."""
    up = lambda x: -(-x // 256) * 256   # noqa: E731
    return K.workspace(up(rows * d * 4) + up(rows * 8))


@pytest.mark.parametrize("lens,hq,hkv,d", [
    (EDGES, 8, 1, 128),                       # 42 workgroups: edges of the shares
    ([1025, 2048, 1793, 3971], 64, 8, 128),   # 128: the most that are spread
    ([1025, 2048, 1793, 3971], 16, 8, 64),
    ([9300, 5, 8193], 4, 2, 128),             # the merge in four wavefronts
    ([69 * 1024 + 7], 2, 1, 64),
    ([65 * 1024], 1, 1, 128),
])
def test_spread_shares_give_the_same_bits(lens, hq, hkv, d):
    """A small batch's shares as workgroups of their own against the least
    workspace, which keeps them together; then with an empty sequence, and ids
    outside the layer, which are skipped though block 0, loaded for them, is NaN."""
    b = _batch(lens, hq, hkv, d, "bf16", seed=215)
    dev = Dev(b)
    say("decode spread", lens, hq, hkv, d)
    rows = len(lens) * hq * -(-max(lens) // 1024)
    least = _least_workspace(rows, d)
    full = K.workspace(K.decode_workspace_bytes(len(lens), hq, d, max(lens)))
    assert full.numel() >= 4 * rows * (d + 2) * 4
    full.view(torch.float32).fill_(float("nan"))
    whole = dev.decode(ws=full)
    assert_parity(whole, oracle_decode(b), "bf16", f"spread {hq}/{hkv}/{d}",
                  seq_bounds(b, decode=True))
    assert torch.equal(whole.view(torch.int16), dev.decode(ws=least).view(torch.int16))
    dev.bt[dev.bt == 0] = -1
    dev.bt[0, 3:37:11] = b.num_blocks
    if len(lens) > 1:
        dev.sl[1] = 0
    dev.kv.view(b.num_blocks, -1)[0] = float("nan")
    some = dev.decode(ws=full)
    assert torch.isfinite(some).all() and (len(lens) == 1 or not some[1].any())
    assert torch.equal(some.view(torch.int16), dev.decode(ws=least).view(torch.int16))


@pytest.mark.parametrize("seqs", [17, 128, 129])   # 136, 1024 and 1032 workgroups
def test_loading_ahead_gives_the_same_bits(seqs):
    """head_dim 64 on both sides of the rules on the number of workgroups: each
    sequence's bits are those of a batch of the same lengths far above them."""
    lens = [EDGES[s % len(EDGES)] for s in range(seqs)]
    b = _batch(lens, 8, 4, 64, "bf16", seed=216)
    dev = Dev(b)
    say("decode ahead", seqs)
    got = dev.decode()
    many = K.decode(dev.q.repeat(10, 1, 1), dev.kv, b.num_blocks, dev.bt.repeat(10, 1),
                    dev.sl.repeat(10), num_kv_heads=4, max_seq_len=b.max_seq_len, scale=b.scale)
    assert torch.equal(got.view(torch.int16), many[:seqs].view(torch.int16))
    assert_parity(got, oracle_decode(b), "bf16", f"ahead {seqs}", seq_bounds(b, decode=True))


@pytest.mark.parametrize("hq,hkv,d,dtype", [(8, 2, 128, "bf16"), (2, 2, 128, "bf16"),
                                            (8, 1, 64, "bf16"), (8, 2, 64, "f32")])
def test_short_contexts_under_any_bound(hq, hkv, d, dtype):
    """Contexts of one share (written without a merge) and of up to four, under
    the bounds at which a call's number of wavefronts changes, spread (2048) and
    not: the same bits as under a bound of two splits that is not spread."""
    lens = [1, 2, 31, 63, 64, 65, 127, 128, 129, 191, 192, 193, 200, 256, 257, 300, 384, 385]
    b = _batch(lens, hq, hkv, d, dtype, seed=217)
    dev = Dev(b)
    dev.bt = torch.nn.functional.pad(dev.bt, (0, 128 - dev.bt.shape[1]), value=-1).contiguous()
    kw = dict(num_kv_heads=hkv, scale=b.scale)
    say("decode short contexts", hq, hkv, d, dtype)
    least = _least_workspace(len(lens) * hq * 2, d)
    want = K.decode(dev.q, dev.kv, b.num_blocks, dev.bt, dev.sl, max_seq_len=2048, ws=least, **kw)
    assert_parity(want, oracle_decode(b), dtype, f"short {hq}/{hkv}/{d}/{dtype}",
                  seq_bounds(b, decode=True))
    as_int = torch.int16 if dtype == "bf16" else torch.int32
    for bound in (64, 65, 128, 129, 192, 193, 300, 385, 1024, 2048):
        n = sum(L <= bound for L in lens)
        got = K.decode(dev.q[:n], dev.kv, b.num_blocks, dev.bt[:n], dev.sl[:n],
                       max_seq_len=bound, **kw)
        assert torch.equal(got.view(as_int), want[:n].view(as_int)), bound


def _loose(dev, copies, bound):
    """Query rows, table and lengths of a batch repeated, under a larger bound."""
    bt = torch.nn.functional.pad(dev.bt, (0, bound // 16 - dev.bt.shape[1]), value=-1)
    return (dev.q.repeat(copies, 1, 1), bt.repeat(copies, 1).contiguous(), dev.sl.repeat(copies))


# 46 (sequence, kv head) pairs of the batch, times splits: four wavefronts, two
# (8280 workgroups), one (16560), and one that takes every 48th split (of 41400)
@pytest.mark.parametrize("hq,hkv,d,dtype", [(8, 2, 128, "bf16"), (2, 2, 128, "bf16"),
                                            (8, 2, 64, "bf16"), (4, 2, 64, "f32")])
@pytest.mark.parametrize("copies,splits", [(1, 178), (1, 180), (4, 90), (15, 60)])
def test_a_loose_bound_gives_the_same_bits(hq, hkv, d, dtype, copies, splits):
    b = _batch(EDGES + [9300, 50 * 1024 - 37], hq, hkv, d, dtype, seed=218)
    dev = Dev(b)
    assert b.num_seqs == 23
    say("decode loose bound", hq, hkv, d, dtype, copies, splits)
    want = dev.decode()
    q, bt, sl = _loose(dev, copies, splits * 1024)
    sl[1] = 0
    got = K.decode(q, dev.kv, b.num_blocks, bt, sl, num_kv_heads=hkv,
                   max_seq_len=splits * 1024, scale=b.scale, out=torch.full_like(q, float("nan")))
    as_int = torch.int16 if dtype == "bf16" else torch.int32
    for c in range(copies):
        part = got[23 * c:23 * (c + 1)].clone()
        if c == 0:
            assert not part[1].any()
            part[1] = want[1]
        assert torch.equal(part.view(as_int), want.view(as_int)), c
    if dtype == "bf16" and d == 128:
        half = b.num_blocks // 2
        flat = dev.kv.view(b.num_blocks, -1)
        two = K.decode_two_tensor(q, flat[:half].contiguous(), half, flat[half:].contiguous(),
                                  b.num_blocks - half, bt, sl, num_kv_heads=hkv,
                                  max_seq_len=splits * 1024, scale=b.scale)
        assert torch.equal(two.view(as_int), got.view(as_int))


def test_fp32_turns_of_short_contexts_give_the_same_bits():
    """1024 workgroups of at most six steps, where two wavefronts take turns,
    against one sequence at a time."""
    lens = [30 + 11 * s for s in range(32)] + [384]
    b = _batch(lens[1:], 4, 2, 64, "f32", seed=219)
    dev = Dev(b)
    say("decode fp32 turns")
    q, bt, sl = _loose(dev, 16, 384)
    got = K.decode(q, dev.kv, b.num_blocks, bt, sl, num_kv_heads=2, max_seq_len=384,
                   scale=b.scale)
    assert_parity(got[:32], oracle_decode(b), "f32", "fp32 turns", seq_bounds(b, decode=True))
    for s in range(0, 32, 5):
        one = K.decode(dev.q[s:s + 1], dev.kv, b.num_blocks, dev.bt[s:s + 1].contiguous(),
                       dev.sl[s:s + 1].contiguous(), num_kv_heads=2, max_seq_len=384,
                       scale=b.scale)
        assert torch.equal(one[0].view(torch.int32), got[480 + s].view(torch.int32)), s


def test_a_loose_bound_costs_little():
    """64 contexts of 30 to 300 tokens under a bound of 131072: the workgroups
    without tokens cost about half of what the others do (16 against 11 us), six
    times that when each held four wavefronts."""
    lens = [30 + (s * 37) % 271 for s in range(64)]
    b = _batch(lens, 32, 8, 128, "bf16", seed=220)
    dev = Dev(b)
    say("decode cost of a loose bound")

    def us(bound):
        q, bt, sl = _loose(dev, 1, bound)
        ws = K.workspace(K.decode_workspace_bytes(64, 32, 128, bound))
        out = torch.empty_like(q)

        def call():
            K.decode(q, dev.kv, b.num_blocks, bt, sl, num_kv_heads=8, max_seq_len=bound,
                     scale=b.scale, out=out, ws=ws)
        for _ in range(20):
            call()
        times = []
        for _ in range(5):
            ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            ev[0].record()
            for _ in range(50):
                call()
            ev[1].record()
            torch.cuda.synchronize()
            times.append(ev[0].elapsed_time(ev[1]) * 20)
        return min(times)

    tight, loose = us(512), us(131072)
    say(f"bound 512 {tight:.1f} us, bound 131072 {loose:.1f} us")
    assert loose < 3 * tight
