"""Hand-out of the attention kernel's work items: every item exactly once, the
workspace left zeroed, for launches that take their items by position only, by
position and through the queues' counters, and (many items per workgroup)
through the counters with helping between queues.

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
])
def test_every_item_once(D, Hq, Hkv, B, q_max, P_max):
    rng = np.random.default_rng(B)
    q_len = rng.integers(1, q_max + 1, B)
    q_len[rng.random(B) < 0.1] = 0        # requests without queries
    q_len[int(rng.integers(B))] = q_max
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
    q = randn(int(cu[-1]), Hq, D)
    scale = D ** -0.5
    cu_d, L_d = torch.from_numpy(cu).cuda(), torch.from_numpy(L).cuda()

    want = torch.zeros_like(q)
    ws = torch.zeros(64, dtype=torch.uint8, device="cuda")
    tiles = -(-q_max * (Hq // Hkv) // 128)
    step = max(1, 256 // (tiles * Hkv))   # requests per small launch: at most 256 items
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
        assert torch.equal(got, want)
        assert int(ws.count_nonzero()) == 0
