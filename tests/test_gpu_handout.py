"""Hand-out of the attention kernel's work items: every item exactly once, the
workspace left zeroed, for launches that take their items by position only, by
position and through the queues' counters, and (many items per workgroup)
through the counters with helping between queues; with few of the item numbers
holding work, which long launches count before they start; and in the wide layout.

The reference is the same batch in small launches of one item per workgroup
(checked against the fp64 oracle elsewhere): a query row meets the same keys in
the same order however the batch is cut, so outputs must be equal bit for bit.
"""
import numpy as np
import pytest
import torch

from paper_2507_08523_amd import ilpc

pytestmark = pytest.mark.gpu

BLOCK = 16


@pytest.mark.parametrize("D,Hq,Hkv,B,q_max,P_max", [
    (128, 8, 2, 31, 365, 96),    # 62 pairs, not a multiple of 8: pieces of items dealt to the queues
    (128, 8, 8, 66, 130, 64),    # just over one item per workgroup (66 x 8 x 2 columns tiles of 128)
    (128, 32, 8, 29, 500, 200),  # ragged, several rounds by position, the rest through the counters
    (128, 8, 8, 1050, 40, 30),   # more than 16 items per workgroup: counters, helping, exit count
    (64, 8, 4, 197, 30, 50),     # head size 64: three workgroups per CU
    (64, 12, 4, 40, 400, 60),
    (64, 4, 1, 12400, 20, 20),
    (128, 32, 8, 80, 700, 200),  # the wide layout: 256-column items
    (128, 28, 4, 150, 600, 60),  # a group of 7
    (128, 64, 8, 700, 32, 0),    # one tile an item
    (128, 64, 8, 336, 64, 12000),  # up to 189 tiles
])
def test_every_item_once(D, Hq, Hkv, B, q_max, P_max):
    rng = np.random.default_rng(B)
    q_len = rng.integers(1, q_max + 1, B)
    q_len[rng.random(B) < 0.1] = 0        # requests without queries
    q_len[int(rng.integers(B))] = q_max
    _check(D, Hq, Hkv, q_len, P_max, rng)


@pytest.mark.parametrize("D,Hq,Hkv,B,long,n_long,short", [
    (128, 8, 8, 64, 2100, 1, 1),     # nearly all numbers empty: fewer items than workgroups by far
    (128, 32, 8, 40, 1300, 2, 40),
    (128, 8, 8, 300, 700, 30, 100),
    (128, 8, 8, 200, 1400, 120, 300),  # still a long launch when counted
    (64, 16, 2, 256, 900, 1, 0),     # one request with queries
    (128, 28, 4, 9, 3600, 1, 1),     # counted for its long pairs on four queues
    (128, 28, 4, 8, 3600, 8, 1),     # and all of them full
    (64, 4, 1, 2047, 330, 9, 3),     # the most requests with one to a group of the count
    (64, 4, 1, 2048, 330, 9, 3),     # two to a group
    (64, 4, 1, 9001, 330, 300, 2),   # eight, the last group short
    (64, 4, 1, 300, 0, 1, 0),        # no query at all
])
def test_numbers_without_work(D, Hq, Hkv, B, long, n_long, short):
    rng = np.random.default_rng(B + long)
    q_len = rng.integers(0, short + 1, B)
    q_len[rng.permutation(B)[:n_long]] = long
    q_len[-1] = long if B % 2 else q_len[-1]
    _check(D, Hq, Hkv, q_len, 40, rng, q_max=long or 1500)


@pytest.mark.parametrize("short", [1, 0])
def test_rows_on_both_sides_of_the_wide_layouts_line(short):
    """Eight 256-column items a CU: as many rows, and one fewer."""
    Hq, B = 32, 64
    line = 8 * 256 * torch.cuda.get_device_properties(0).multi_processor_count // Hq
    q_len = np.full(B, (line - 512) // (B - 1))
    q_len[7] = 512                       # 64 x 8 x 16 numbers: a long launch
    q_len[9] += line - q_len.sum() - short
    assert q_len.sum() == line - short
    _check(128, Hq, 8, q_len, 300, np.random.default_rng(short), q_max=512)


def _check(D, Hq, Hkv, q_len, P_max, rng, q_max=None):
    B = len(q_len)
    q_max = q_max or int(q_len.max())
    P = rng.integers(0, P_max + 1, B)
    L = (P + q_len).astype(np.int32)
    L = np.maximum(L, 1).astype(np.int32)
    mb = -(-int(L.max()) // BLOCK)
    NB = 512
    gen = torch.Generator(device="cuda")
    gen.manual_seed(B)

    def randn(*shape):
        return torch.randn(shape, generator=gen, device="cuda", dtype=torch.bfloat16)

    k_pool, v_pool = randn(NB, Hkv, BLOCK, D), randn(NB, Hkv, D, BLOCK)
    tables = torch.from_numpy(rng.integers(0, NB, (B, mb)).astype(np.int32)).cuda()
    cu = np.zeros(B + 1, np.int32)
    cu[1:] = np.cumsum(q_len)
    q = randn(max(int(cu[-1]), 1), Hq, D)
    scale = D ** -0.5
    cu_d, L_d = torch.from_numpy(cu).cuda(), torch.from_numpy(L).cuda()

    want = torch.zeros_like(q)
    ws = torch.zeros(64, dtype=torch.uint8, device="cuda")
    tiles = -(-q_max * (Hq // Hkv) // 128)
    step = max(1, 256 // (tiles * Hkv))   # requests per small launch: at most 256 items, or one request
    for a in range(0, B, step):
        e = min(a + step, B)
        rows = slice(int(cu[a]), int(cu[e]))
        if cu[e] == cu[a]:
            continue
        sub = torch.from_numpy((cu[a:e + 1] - cu[a]).astype(np.int32)).cuda()
        ilpc.paged_prefill_attn(q[rows], k_pool, v_pool, tables[a:e], sub, L_d[a:e].clone(), q_max, scale,
                                want[rows], ws)
    assert torch.isfinite(want).all()
    for _ in range(2):                     # twice on one workspace: the counters must be left zero
        got = torch.full_like(q, float("nan"))
        ilpc.paged_prefill_attn(q, k_pool, v_pool, tables, cu_d, L_d, q_max, scale, got, ws)
        torch.cuda.synchronize()
        assert torch.equal(got[:int(cu[-1])], want[:int(cu[-1])])
        assert int(ws.count_nonzero()) == 0


@pytest.mark.parametrize("D,Hq,Hkv,B,shared,q_max", [
    (128, 32, 8, 512, 256, 128),   # one launch
    (64, 16, 4, 700, 192, 60),
    (128, 32, 8, 300, 96, 128),    # two launches: less than three shared tiles
    (64, 16, 4, 900, 160, 70),
])
def test_shared_split_without_work(D, Hq, Hkv, B, shared, q_max):
    """The split at a shared prefix, nearly all of whose numbers are empty, twice on
    one workspace: close to the single pass, the counters left zero."""
    rng = np.random.default_rng(B)
    q_len = rng.integers(0, 4, B)
    q_len[int(rng.integers(B))] = q_max
    L = (shared + rng.integers(0, 30, B) + q_len).astype(np.int32)
    mb, NB = -(-int(L.max()) // BLOCK), 256
    gen = torch.Generator(device="cuda").manual_seed(B)
    randn = lambda *s: torch.randn(s, generator=gen, device="cuda", dtype=torch.bfloat16)  # noqa: E731
    k_pool, v_pool = randn(NB, Hkv, BLOCK, D), randn(NB, Hkv, D, BLOCK)
    tables = rng.integers(0, NB, (B, mb)).astype(np.int32)
    tables[:, :shared // BLOCK] = tables[0, :shared // BLOCK]
    cu = np.concatenate([[0], np.cumsum(q_len)]).astype(np.int32)
    q = randn(int(cu[-1]), Hq, D)
    dev = [torch.from_numpy(x).cuda() for x in (tables, cu, L)]
    want = torch.full_like(q, float("nan"))
    ilpc.paged_prefill_attn(q, k_pool, v_pool, *dev, q_max, D ** -0.5, want,
                            torch.zeros(64, dtype=torch.uint8, device="cuda"))
    ws = torch.zeros(ilpc.attn_cascade_workspace_bytes(B, q_max, Hq, Hkv, D), dtype=torch.uint8, device="cuda")
    for _ in range(2):
        got = torch.full_like(q, float("nan"))
        ilpc.paged_prefill_attn_cascade(q, k_pool, v_pool, *dev, q_max, shared, D ** -0.5, got, ws)
        torch.cuda.synchronize()
        # |V| reaches about 4.5; both sides round the probabilities and the output to
        # bf16 (2^-9 relative each): 2 * 4.5 * 2^-8 = 3.5e-2 bounds the difference
        assert float((got.float() - want.float()).abs().max()) <= 3.5e-2
        assert int(ws[:128].count_nonzero()) == 0


def test_one_long_request_among_short_ones_costs_its_own_work():
    """64 requests, one of 4000 new tokens: the two parts by themselves take as long
    together (measured: 1.1 times; with all numbers handed out one by one 5 times)."""
    Hq, Hkv, D, B, long = 32, 8, 128, 64, 4000
    q_len = np.ones(B, np.int64)
    q_len[20] = long
    us = []
    for part in (q_len, q_len[20:21], np.delete(q_len, 20)):
        L = (part + 256).astype(np.int32)
        n, mb = len(part), -(-int(L.max()) // BLOCK)
        nb = -(-L // BLOCK)
        tables = np.zeros((n, mb), np.int32)
        for r in range(n):
            tables[r, :nb[r]] = np.arange(nb[r]) + nb[:r].sum()
        k_pool = torch.randn(int(nb.sum()), Hkv, BLOCK, D, device="cuda", dtype=torch.bfloat16)
        v_pool = torch.randn(int(nb.sum()), Hkv, D, BLOCK, device="cuda", dtype=torch.bfloat16)
        cu = np.concatenate([[0], np.cumsum(part)]).astype(np.int32)
        q = torch.randn(int(cu[-1]), Hq, D, device="cuda", dtype=torch.bfloat16)
        out = torch.empty_like(q)
        dev = [torch.from_numpy(x).cuda() for x in (tables, cu, L)]
        ws = torch.zeros(ilpc.attn_workspace_bytes(n, int(part.max()), Hq, Hkv, D), dtype=torch.uint8, device="cuda")
        times = []
        for _ in range(9):
            ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            ev[0].record()
            for _ in range(10):
                ilpc.paged_prefill_attn(q, k_pool, v_pool, *dev, int(part.max()), D ** -0.5, out, ws)
            ev[1].record()
            torch.cuda.synchronize()
            times.append(ev[0].elapsed_time(ev[1]) * 100)
        us.append(sorted(times)[4])
    print(f"[hand-out] mixed {us[0]:.1f} us, long {us[1]:.1f}, short {us[2]:.1f}", flush=True)
    assert us[0] <= 1.6 * (us[1] + us[2])
