"""Planned prefill steps: tiles whose keys are shared by several workgroups and
merged, items ordered over sequences, one-row sequences beside tiles. Against the
oracle on every row, with the kernels launched and what the plan shares, and the
same call with a workspace that only holds the list of whole tiles."""
import pytest
import torch

import paper_2608_23658_amd.kvattn as K
from workloads import make_batch_from_lens
from tests.gpu_helpers import (seq_bounds, Dev, assert_parity, oracle_prefill, require_gpu, say)

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def _list_bytes(b):
    """The least workspace a call takes: 8 bytes per tile of 32 rows."""
    return ((b.total_q_tokens // 32 + b.num_seqs + 1) * 8 + 16 + 255) // 256 * 256


def _kernels(call):
    with K.KernelTrace(8) as tr:
        call()
    torch.cuda.synchronize()
    return tr.names


def _plan_head(ws):
    """Items, shared tiles and shared one-row sequences of the call that used ws."""
    torch.cuda.synchronize()
    return tuple(ws[:12].view(torch.int32).tolist())


MAP = ["prefill_tile_map", "prefill"]
PLAN = ["prefill_plan", "prefill"]
MERGE = PLAN + ["prefill_combine"]


def _check(L, N, hq, hkv, seed, names, shared=False, shared_rows=0):
    """Against the oracle, with the kernels the call launches, whether the plan
    shares tiles and how many one-row sequences it shares (None: some)."""
    b = make_batch_from_lens(L, N, dtype="bf16", num_q_heads=hq, num_kv_heads=hkv,
                             head_dim=128, block_size=16, seed=seed)
    d = Dev(b)
    ws = K.workspace(K.prefill_workspace_bytes(b.num_seqs, b.total_q_tokens, hq, 128))
    ws.fill_(0xff)                     # no initial contents are needed
    say("prefill planned", L[:4], N[:4], hq, hkv)
    ref = oracle_prefill(b)
    for what, w, kernels in (("planned", ws, names), ("planned again", ws, names),
                             ("whole tiles", K.workspace(_list_bytes(b)), MAP)):
        assert w is ws or w.numel() < ws.numel()
        out = torch.full_like(d.q, float("nan"))
        assert _kernels(lambda: d.prefill(ws=w, out=out)) == kernels, what
        if kernels is not MAP:
            _, splits, row_splits = _plan_head(w)
            assert (splits > 0) == shared, (what, splits)
            assert row_splits == shared_rows if shared_rows is not None else row_splits > 0, what
        assert_parity(out, ref, "bf16", f"{what} {hq}/{hkv}", seq_bounds(b))


# 16 pieces of one tile; pieces that do not divide the steps; the last tile of
# one row; a length that ends inside a block; a sequence too short to share
@pytest.mark.parametrize("hq,hkv", [(8, 1), (4, 1), (2, 1), (1, 1), (12, 3), (32, 8), (64, 8)])
def test_shared_tiles(hq, hkv):
    _check([4096, 2111, 640, 70], [33, 65, 200, 9], hq, hkv, 301, MERGE, shared=True)


@pytest.mark.parametrize("hq,hkv", [(32, 8), (8, 8)])
def test_one_short_chunk_over_a_long_context(hq, hkv):
    _check([6351], [201], hq, hkv, 302, MERGE, shared=True)


def test_more_sequences_than_one_planning_pass_holds():
    n = [1 + s % 3 for s in range(1100)]
    _check([x + s % 130 for s, x in enumerate(n)], n, 4, 1, 303, PLAN)


def test_more_tiles_than_threads_plan_at_once():
    _check([17600, 900], [17600, 700], 8, 1, 304, MERGE)


def test_rows_shared_in_several_planning_passes():
    """One-row sequences long enough to be shared in each of the plan's passes of
    512 sequences, among short ones and a chunk of more rows."""
    L = [1 + (s * 7) % 120 for s in range(1100)]
    n = [1] * 1100
    for s, x in ((10, 3000), (511, 4000), (512, 1025), (700, 9000), (1099, 5000)):
        L[s] = x
    L[520], n[520] = 900, 200
    _check(L, n, 4, 1, 313, MERGE, shared_rows=5)


# one-row sequences: shared by several items, up to a split's edges, one token;
# alone (rows only), one single row, and next to tiles
@pytest.mark.parametrize("hq,hkv", [(8, 1), (4, 4), (16, 8), (12, 3), (32, 8)])
@pytest.mark.parametrize("tiles", [False, True])
def test_one_row_sequences(hq, hkv, tiles):
    L = [9000, 1, 63, 512, 513, 1024, 1025, 4097] + ([2500, 300] if tiles else [])
    _check(L, [1] * 8 + ([130, 3] if tiles else []), hq, hkv, 306, MERGE, shared=tiles,
           shared_rows=3)


# both sides of the rules by which a call may share tiles (16 steps with the chip
# nearly idle are 15.4 of it) and one-row sequences (2048 tokens)
@pytest.mark.parametrize("L,N,hq,hkv,names,shared_rows", [
    ([1024], [300], 8, 1, MAP, 0), ([1025], [300], 8, 1, MERGE, 0),
    ([1100, 2048], [1100, 1], 32, 8, PLAN, 0), ([1100, 2049], [1100, 1], 32, 8, MERGE, 1)])
def test_share_rule_edges(L, N, hq, hkv, names, shared_rows):
    _check(L, N, hq, hkv, 309, names, shared=L == [1025], shared_rows=shared_rows)


def test_a_single_row():
    _check([5000], [1], 8, 2, 307, MERGE, shared_rows=1)


def test_a_one_row_sequence_without_context_gives_zeros():
    b = make_batch_from_lens([40, 600, 17], [1, 1, 17], dtype="bf16", num_q_heads=8,
                             num_kv_heads=2, head_dim=128, block_size=16, seed=308)
    d = Dev(b)
    d.sl[0] = 0
    say("prefill one row, length 0")
    out = d.prefill(out=torch.full_like(d.q, float("nan")))
    assert (out[0] == 0).all()
    ref = oracle_prefill(b)
    assert_parity(out[1:], ref[1:], "bf16", "rows after an empty one")


def test_a_workspace_below_the_tile_list_is_refused():
    b = make_batch_from_lens([900], [300], dtype="bf16", num_q_heads=8, num_kv_heads=2,
                             head_dim=128, block_size=16, seed=305)
    with pytest.raises(K.KvAttnError) as e:
        Dev(b).prefill(ws=torch.empty(_list_bytes(b) - 1, dtype=torch.uint8, device="cuda"))
    assert e.value.code == K.KV_ERR_INVALID


def test_a_plan_of_several_passes_launches_no_merge_for_tiles():
    """600 one-row sequences of up to 1500 tokens: the plan shares no tiles above
    512 sequences, and one-row ones only from 2048 tokens on, so nothing can
    leave partials."""
    n = [1] * 600
    b = make_batch_from_lens([1 + (s * 7) % 120 for s in range(599)] + [1500], n, dtype="bf16",
                             num_q_heads=4, num_kv_heads=1, head_dim=128, block_size=16, seed=310)
    d = Dev(b)
    say("prefill several passes, no merge")
    out = {}
    names = _kernels(lambda: out.update(o=d.prefill()))
    assert names == ["prefill_plan", "prefill"], names
    assert_parity(out["o"], oracle_prefill(b), "bf16", "600 rows", seq_bounds(b))


# tiles and one-row sequences that fit one round, at its edge (32 workgroups'
# worth at 8 kv heads), and one more; sequences without new rows among them
@pytest.mark.parametrize("rows", [5, 26, 27])
@pytest.mark.parametrize("hq,hkv", [(32, 8), (8, 8)])
def test_one_round_of_tiles_and_one_row_sequences(rows, hq, hkv):
    R = 32 * 8 * hkv // hq
    L = [2 * R + 70, 40, R] + [3 + 29 * s for s in range(rows)] + [9]
    n = [2 * R + 1, 0, R] + [1] * rows + [2]
    b = make_batch_from_lens(L, n, dtype="bf16", num_q_heads=hq, num_kv_heads=hkv, head_dim=128,
                             block_size=16, seed=311)
    assert b.max_seq_len <= 1024
    d = Dev(b)
    ws = K.workspace(K.prefill_workspace_bytes(b.num_seqs, b.total_q_tokens, hq, 128))
    ws.fill_(0xff)
    say("prefill one round", rows, hq, hkv)
    out = d.prefill(ws=ws, out=torch.full_like(d.q, float("nan")))
    assert _plan_head(ws) == (5 + rows, 0, 0)
    assert_parity(out, oracle_prefill(b), "bf16", f"one round {rows} {hq}/{hkv}", seq_bounds(b))


# whether tiles are shared under a bound far above the lengths: too short to
# share, walks that gain little, and ones that gain (10 steps of idle chip)
@pytest.mark.parametrize("L,N,hq,hkv,shared", [([200], [200], 32, 8, False),
                                               ([70, 90, 100], [64, 50, 100], 32, 8, False),
                                               ([768, 300, 20], [512, 1, 1], 32, 8, False),
                                               ([1280], [1024], 32, 8, True),
                                               ([768, 90], [40, 1], 4, 1, True)])
def test_a_loose_bound_shares_by_the_lengths(L, N, hq, hkv, shared):
    b = make_batch_from_lens(L, N, dtype="bf16", num_q_heads=hq, num_kv_heads=hkv, head_dim=128,
                             block_size=16, seed=312)
    d = Dev(b)
    bt = torch.nn.functional.pad(d.bt, (0, 8192 - d.bt.shape[1]), value=-1).contiguous()
    ws = K.workspace(K.prefill_workspace_bytes(b.num_seqs, b.total_q_tokens, hq, 128))
    ws.fill_(0xff)
    say("prefill loose bound", L, N)
    out = K.prefill_chunk(d.q, d.kv, b.num_blocks, bt, d.sl, d.cu, num_kv_heads=hkv,
                          max_seq_len=131072, scale=b.scale, ws=ws,
                          out=torch.full_like(d.q, float("nan")))
    items, splits, row_splits = _plan_head(ws)
    R = 32 * 8 * hkv // hq
    whole = sum(-(-n // R) if n > 1 else 1 for n in N)
    assert (splits > 0) == shared and row_splits == 0
    assert items > whole if shared else items == whole
    assert_parity(out, oracle_prefill(b), "bf16", "loose bound", seq_bounds(b))


def test_the_least_workspace_gives_a_sequences_own_bits():
    """With room for the list of whole tiles only, a row's bits depend on its own
    sequence: alone under its own length as the bound, or in a batch under a
    larger one, one-row sequences included."""
    L, N = [4096, 2111, 9000, 640, 70, 300], [33, 65, 1, 200, 9, 1]
    b = make_batch_from_lens(L, N, dtype="bf16", num_q_heads=8, num_kv_heads=2, head_dim=128,
                             block_size=16, seed=314)
    d = Dev(b)
    ws = K.workspace(_list_bytes(b))
    say("prefill least workspace")
    whole = d.prefill(ws=ws)
    assert_parity(whole, oracle_prefill(b), "bf16", "least workspace", seq_bounds(b))
    for s in range(len(L)):
        lo, hi = int(b.cu_seqlens_q[s]), int(b.cu_seqlens_q[s + 1])
        cu = torch.tensor([0, hi - lo], dtype=torch.int32, device="cuda")
        one = K.prefill_chunk(d.q[lo:hi], d.kv, b.num_blocks, d.bt[s:s + 1].contiguous(),
                              d.sl[s:s + 1].contiguous(), cu, num_kv_heads=2, max_seq_len=L[s],
                              scale=b.scale, ws=ws)
        assert torch.equal(one.view(torch.int16), whole[lo:hi].view(torch.int16)), s


def test_beside_four_rounds_of_tiles_rows_are_shared_and_tiles_are_not():
    """1024 workgroups of tiles: their rows have the bits of whole tiles; a one-row
    sequence above 8192 tokens is shared all the same."""
    b = make_batch_from_lens([4096, 9000, 700], [4096, 1, 1], dtype="bf16", num_q_heads=64,
                             num_kv_heads=8, head_dim=128, block_size=16, seed=315)
    d = Dev(b)
    ws = K.workspace(K.prefill_workspace_bytes(b.num_seqs, b.total_q_tokens, 64, 128))
    say("prefill four rounds")
    out = torch.empty_like(d.q)
    assert _kernels(lambda: d.prefill(ws=ws, out=out)) == MERGE
    assert _plan_head(ws)[1:] == (0, 1)
    least = d.prefill(ws=K.workspace(_list_bytes(b)))
    assert torch.equal(out[:4096].view(torch.int16), least[:4096].view(torch.int16))
    ref = oracle_prefill(b, seqs=[1, 2])
    assert_parity(out[4096:], ref[4096:], "bf16", "rows beside four rounds", [0, 1, 2])
