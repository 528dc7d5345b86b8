"""A row's result does not depend on how many rows share the call: products take
their tiles by the number of rows, and every tile adds in the same order, so a
sequence alone and the same sequence in larger batches give the same bits."""

from __future__ import annotations

import pytest

from tests.gpu_util import log, need_gpu
from tests.test_gpu_sweep import _check
from workloads import MODELS

pytestmark = pytest.mark.gpu

BASE = dict(n_layers=1, rope_theta=10000.0, norm_eps=1e-6, init_std=0.05, lm_head_scale=1.0, vocab=300, mask_id=299)
DENSE = dict(BASE, n_experts=0, top_k=0, expert_ffn_dim=0, n_shared_experts=0)

SHAPES = {
    # d_model below and at the length from which 256x256 tiles are taken, head
    # widths 64 and 128 (the order of the QKV rows), dense and expert FFNs
    "dense_hd64": dict(DENSE, d_model=256, n_heads=4, n_kv_heads=2, head_dim=64, ffn_dim=320),
    "dense_hd128_wide": dict(DENSE, d_model=2048, n_heads=16, n_kv_heads=2, head_dim=128, ffn_dim=2112),
    "moe_hd128": dict(BASE, d_model=256, n_heads=2, n_kv_heads=1, head_dim=128, ffn_dim=0, n_experts=24, top_k=3,
                      expert_ffn_dim=192, n_shared_experts=1),
    "moe_hd64_no_shared": dict(BASE, d_model=384, n_heads=6, n_kv_heads=2, head_dim=64, ffn_dim=0, n_experts=5,
                               top_k=1, expert_ffn_dim=64, n_shared_experts=0),
    # logit rows longer than what the expert products write (partial logits go elsewhere)
    "moe_256_narrow": dict(BASE, d_model=128, n_heads=2, n_kv_heads=2, head_dim=64, ffn_dim=0, n_experts=256, top_k=1,
                           expert_ffn_dim=64, n_shared_experts=0),
    "moe_130": dict(BASE, d_model=512, n_heads=4, n_kv_heads=2, head_dim=64, ffn_dim=0, n_experts=130, top_k=8,
                    expert_ffn_dim=64, n_shared_experts=1),
}


@pytest.mark.parametrize("name", list(SHAPES))
@pytest.mark.parametrize("seq", [1, 37, 130])
def test_rows_do_not_depend_on_the_batch(name, seq):
    need_gpu()
    import torch
    from paper_2608_02625_amd import Refiner
    shape = SHAPES[name]
    r = Refiner(shape, 7)
    d = shape["d_model"]
    top = max(2, (9000 if d < 1024 else 4500) // seq)
    g = torch.Generator().manual_seed(seq)
    x = torch.randn(top * seq, d, generator=g).cuda()
    ref = r.debug_layer(0, x[:seq].clone(), 1, seq)
    assert torch.isfinite(ref).all()
    batches = sorted({b for b in (2, 3, 300 // seq, 700 // seq, 1500 // seq, 2600 // seq, 4400 // seq, top) if 1 < b <= top})
    for b in batches:
        y = r.debug_layer(0, x[:b * seq].clone(), b, seq)
        assert torch.equal(y[:seq], ref), f"batch {b}"
        lone = r.debug_layer(0, x[(b - 1) * seq:b * seq].clone(), 1, seq)
        assert torch.equal(y[-seq:], lone), f"last row of batch {b}"
    log(f"[tiles {name} seq {seq}] batches {batches} equal the sequence alone")


@pytest.mark.parametrize("over,seq,batch", [
    # row counts that put O, dense down, QKV and gate/up on 256x256 tiles: K 2048
    # in one round, K 1024 and 512 in several, and partly filled row tiles
    (dict(d_model=2048, n_heads=16, n_kv_heads=4, head_dim=128, ffn_dim=2112), 64, 128),
    (dict(d_model=1024, n_heads=16, n_kv_heads=4, head_dim=64, ffn_dim=4096), 64, 512),
    (dict(d_model=1024, n_heads=8, n_kv_heads=2, head_dim=128, ffn_dim=3072), 61, 540),
    (dict(d_model=512, n_heads=8, n_kv_heads=8, head_dim=64, ffn_dim=1024), 64, 1024),
    # gate/up with fewer K tiles than stages
    (dict(d_model=128, n_heads=4, n_kv_heads=2, head_dim=64, ffn_dim=1024), 64, 1024),
])
def test_rows_of_large_calls(over, seq, batch):
    """The same at the largest tiles: sequences of a large call equal the
    sequence alone, bit for bit."""
    need_gpu()
    import torch
    from paper_2608_02625_amd import Refiner
    r = Refiner(dict(DENSE, **over), 5)
    x = torch.randn(batch * seq, over["d_model"], generator=torch.Generator().manual_seed(batch)).cuda()
    y = r.debug_layer(0, x.clone(), batch, seq)
    for b in (0, 1, batch // 2, batch - 2, batch - 1):
        lone = r.debug_layer(0, x[b * seq:(b + 1) * seq].clone(), 1, seq)
        assert torch.equal(y[b * seq:(b + 1) * seq], lone), f"sequence {b}"


@pytest.mark.parametrize("over,B,P,D", [
    # router with 2, 4 and 8 K parts, 2 and 4 expert blocks of 64, few and many tokens per group
    (dict(d_model=128, n_heads=2, n_kv_heads=2, head_dim=64, n_experts=256, top_k=1, expert_ffn_dim=64,
          n_shared_experts=0), 2, 3, 30),
    (dict(d_model=640, n_heads=5, n_kv_heads=5, head_dim=128, n_experts=130, top_k=8, expert_ffn_dim=64,
          n_shared_experts=1), 1, 40, 25),
    (dict(d_model=768, n_heads=6, n_kv_heads=2, head_dim=128, n_experts=65, top_k=3, expert_ffn_dim=128,
          n_shared_experts=1), 1, 0, 65),
    (dict(d_model=512, n_heads=4, n_kv_heads=2, head_dim=64, n_experts=200, top_k=8, expert_ffn_dim=64,
          n_shared_experts=0), 5, 100, 333),
])
def test_router_against_the_oracle(over, B, P, D):
    _check(MODELS["tiny"].replace(n_layers=1, ffn_dim=0, vocab=500, **over), B, P, D, 91, f"router {over['n_experts']}")


@pytest.mark.parametrize("experts,blocks,B,P,D", [
    (256, 2, 2, 3, 30), (256, 3, 1, 0, 37), (200, 2, 2, 7, 30), (200, 3, 3, 60, 70), (129, 2, 1, 1, 96),
])
def test_narrow_experts_over_several_blocks(experts, blocks, B, P, D):
    """Logit rows longer than an expert row pair, in a model of several blocks
    with sequences that end inside a 32-key tile: what the router leaves behind
    must not show in the next block's attention, whatever the workspace held."""
    shape = MODELS["tiny"].replace(n_layers=blocks, d_model=128, n_heads=2, n_kv_heads=2, head_dim=64, ffn_dim=0,
                                   n_experts=experts, top_k=1, expert_ffn_dim=64, n_shared_experts=0, vocab=500)
    assert (P + D) % 32 != 0 and 2 * (shape.expert_ffn_dim + shape.d_model) < 4 * experts
    _check(shape, B, P, D, 17, f"narrow {experts}", workspace_fill=255)


@pytest.mark.parametrize("experts,shared", [(3, 0), (8, 1)])
def test_rows_of_every_expert_tile_height(experts, shared):
    """With top-k = E every expert gets every row: the row counts walk over the
    heights of the expert tiles (steps of 32 rows, one to five tiles), and each
    row must equal what it gets in a small batch."""
    need_gpu()
    import torch
    from paper_2608_02625_amd import Refiner
    shape = dict(BASE, d_model=512, n_heads=4, n_kv_heads=2, head_dim=64, ffn_dim=0, n_experts=experts, top_k=experts,
                 expert_ffn_dim=320, n_shared_experts=shared)
    r = Refiner(shape, 3)
    x = torch.randn(1300, 512, generator=torch.Generator().manual_seed(5)).cuda()
    ref = torch.cat([r.debug_layer(0, x[i:i + 26].clone(), 26, 1) for i in range(0, 1300, 26)])
    for t in (1, 2, 32, 33, 64, 65, 72, 73, 128, 129, 160, 161, 191, 193, 224, 225, 255, 256, 257, 288, 289, 320, 449,
              512, 513, 545, 768, 769, 1024, 1025, 1300):
        y = r.debug_layer(0, x[:t].clone(), t, 1)
        assert torch.equal(y, ref[:t]), f"{t} rows"
    log(f"[expert tile heights E {experts} shared {shared}] equal")
