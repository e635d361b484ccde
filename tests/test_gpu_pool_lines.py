"""A slot pool that starts inside a 128-byte line: two slots share a line there, and a launch that fills one slot while it reads
the other would find old bytes in it.  Such a pool takes the chain of kernels, whatever form is asked for."""
import pytest
import torch

from paper_2605_18071_amd import workloads as W
from tests.test_gpu_parity import small

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from tests import gpu_rig as R


@pytest.mark.parametrize("page,mb,shift", [(16, -1, 16), (16, 0, 64), (8, -1, 112), (4, 0, 48), (64, -1, 32)])
def test_slots_that_share_lines_take_the_chain(page, mb, shift):
    w = small("pool-lines", page=page, ctx=page * 300, topk_pages=24, capacity=36, batch=2, n_kv_heads=2, n_q_heads=4, heavy_count=3,
              n_layers=2, steps=3, rho=0.5)
    rig, chain = R.Rig(w, micro_batches=mb), R.Rig(w, micro_batches=1)
    assert rig.kvd.step_form() == -1
    room = torch.zeros(rig.pool.numel() + 64, dtype=w.torch_dtype, device=R.DEV)
    assert room.data_ptr() % 128 == 0
    shifted = room[shift // 2:shift // 2 + rig.pool.numel()].view(rig.pool.shape)
    rig.kvd.bind_slot_pool(shifted)
    rig.warm()
    rig.kvd.set_step_form(mb)                              # accepted: another pool may be bound
    assert rig.kvd.step_form() == 1
    for r in (rig, chain):
        r.kvd.set_wait_limit_us(0)                         # a step with waits inside would give up
    a, b = (torch.empty((w.n_layers, w.batch, w.n_q_heads, w.head_dim), dtype=torch.float32, device=R.DEV) for _ in range(2))
    qs = list(W.query_stream(w, rig.q0, 2 * w.steps, R.DEV))
    for t in range(w.steps):
        for l in range(w.n_layers):
            rig.step(l, 2 * t, qs[2 * t][l])
            chain.step(l, 2 * t, qs[2 * t][l])
            for what in ("sel_pages", "sel_slots", "counts", "out", "lse"):
                assert torch.equal(getattr(rig, what), getattr(chain, what)), (what, t, l)
        rig.kvd.step_layers(0, w.n_layers, 2 * t + 1, qs[2 * t + 1], a)
        chain.kvd.step_layers(0, w.n_layers, 2 * t + 1, qs[2 * t + 1], b)
        torch.cuda.synchronize()
        assert torch.equal(a, b) and torch.equal(shifted, chain.pool), t
    # a pool that starts on a line: the one launch again
    rig.kvd.set_wait_limit_us(2_000_000)
    rig.kvd.bind_slot_pool(rig.pool)
    rig.warm()
    chain.warm()
    assert rig.kvd.step_form() == -1
    for t in range(w.steps):
        rig.step(0, 10 + t, qs[t][0])
        chain.step(0, 10 + t, qs[t][0])
        assert torch.equal(rig.sel_slots, chain.sel_slots) and float((rig.out - chain.out).norm() / chain.out.norm()) < 1e-3
    rig.close()
    chain.close()
