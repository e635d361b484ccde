"""Where the split-K rule changes: a split keeps whole pages, none is empty, what kvd_set_step_shape took before it still
takes, and the outputs do not depend on the split (against one split, up to the order of the fp32 sums)."""
import pytest
import torch

from paper_2605_18071_amd import kvd as K
from tests import helpers as H
from tests.test_gpu_parity import small

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from tests import gpu_rig as R


@pytest.mark.parametrize("kw,rule,most", [
    (dict(ctx=16 * 300, topk_pages=31, capacity=40), 1, 2),              # 31 tiles: too few for a tile per wave
    (dict(ctx=16 * 300, topk_pages=32, capacity=40), 4, 8),              # 32
    (dict(ctx=16 * 600, topk_pages=256, capacity=300), 16, 32),          # 256 tiles: the most splits before 32 tiles each
    (dict(ctx=16 * 2000, topk_pages=1024, capacity=1100), 32, 64),       # 1024 tiles
    (dict(ctx=64 * 100, page=64, topk_pages=21, capacity=30), 5, 10),    # 84 tiles in 21 pages
])
def test_rule_and_limits(kw, rule, most):
    w = small("split-rule", **{**dict(batch=1, n_kv_heads=4, n_q_heads=8, heavy_count=3, steps=2), **kw})
    rig, one = R.Rig(w, micro_batches=-1), R.Rig(w, micro_batches=-1, attn_splits=max(1, -(-w.topk_pages // 512)))
    assert rig.kvd.step_shape()[2] == rule
    rig.kvd.set_step_shape(attn_splits=most)                            # accepted
    rig.kvd.set_step_shape()
    for t, q in enumerate(R.W.query_stream(w, rig.q0, w.steps, R.DEV)):
        rig.step(0, t, q[0])
        one.step(0, t, q[0])
        assert torch.equal(rig.sel_pages, one.sel_pages)
        # (the probabilities that multiply V keep 16 bits, relative to each split's own maximum)
        assert H.attn_rel_err(rig.n_out.reshape(-1, 128), one.n_out.reshape(-1, 128)) <= 2.0 ** -14
    rig.close()
    one.close()


def test_the_shape_reported_for_several_layers_is_that_of_the_longest_launch():
    """16 units of 1024 pages: eight layers' chunks fill the compute units (two passes per chunk), two layers' do not."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    w, two = (small("shape-query", ctx=16 * 1024, topk_pages=16, capacity=20, batch=4, n_kv_heads=4, n_q_heads=4, n_layers=n,
                    physical_layers=1, heavy_count=2) for n in (8, 2))
    rig, one, short = R.Rig(w, micro_batches=-1), R.Rig(w, micro_batches=-1), R.Rig(two, micro_batches=-1)
    chunks = lambda passes: -(-1024 // (512 * passes))                   # per unit
    for r, passes in ((rig, 2), (short, 1)):
        assert (r.w.n_layers * r.w.units * chunks(1) >= 0.75 * cus) == (passes == 2)
        assert r.kvd.step_shape(multi_layer=True)[:2] == (passes, r.w.units * chunks(passes))
        assert r.kvd.step_shape()[0] == 1
    # a launch of two of the eight layers gives what the layers give one by one
    for t, q in enumerate(R.W.query_stream(w, rig.q0, 2, R.DEV)):
        out = torch.empty((2, w.batch, w.n_q_heads, w.head_dim), dtype=torch.float32, device=R.DEV)
        rig.kvd.step_layers(0, 2, t, q[:2].contiguous(), out)
        for l in range(2):
            one.step(l, t, q[l])
            assert torch.equal(out[l], one.out)
    for r in (rig, one, short):
        r.close()


@pytest.mark.parametrize("units,k,page,most", [
    (128, 512, 16, 16),         # 512 tiles: two splits of 64 tiles each, whatever the number of units
    (140, 289, 256, 64),        # 4624 tiles: as many as there are at most
    (30, 56, 256, 28),
])
def test_units_of_many_pages_take_twice_a_split_per_64_tiles(units, k, page, most):
    ctx = K.Kvd(n_layers=1, batch=units, n_q_heads=4, n_kv_heads=1, page_size=page, max_pages=8200, topk_pages=k,
                capacity_max=k + 8, kv_dtype=torch.bfloat16, micro_batches=-1)
    assert ctx.step_form() == -1
    ctx.set_step_shape(attn_splits=most)
    assert ctx.step_shape()[2] == most
    with pytest.raises(K.KvdError):
        ctx.set_step_shape(attn_splits=most + 1)
    ctx.close()


def test_shapes_of_several_layers_are_taken_whatever_the_form():
    """251 units: the stand-alone attention kernel has one split of 691 pages, more than a workgroup of the one-launch step
    stages; what is set for launches of several layers has that step's two splits in every form of the context."""
    ctx = K.Kvd(n_layers=2, batch=251, n_q_heads=2, n_kv_heads=1, page_size=16, max_pages=800, topk_pages=691, capacity_max=700,
                kv_dtype=torch.bfloat16)
    assert ctx.step_form() == -1
    for form in (0, -1, 1, 2):
        ctx.set_step_form(form)
        for multi in (False, True):
            ctx.set_step_shape(multi_layer=multi)
            assert ctx.step_shape(multi_layer=multi)[2] == 2
            ctx.set_step_shape(passes=2, multi_layer=multi)
            assert ctx.step_shape(multi_layer=multi)[0] == 2
    ctx.close()


def test_a_reported_shape_of_several_layers_gives_the_same_launch_when_it_is_set():
    """8 layers of 16 units with 16 splits, of which a workgroup takes several (9.3 us a layer, 12.3 with a workgroup each)."""
    w = small("shape-again", ctx=16 * 1024, topk_pages=256, capacity=280, batch=4, n_kv_heads=4, n_q_heads=8, n_layers=8,
              physical_layers=1, heavy_count=3)
    rig = R.Rig(w, micro_batches=-1)
    q = next(R.W.query_stream(w, rig.q0, 1, R.DEV)).contiguous()
    outs = [torch.empty((8, w.batch, w.n_q_heads, w.head_dim), dtype=torch.float32, device=R.DEV) for _ in range(3)]
    rig.kvd.step_layers(0, 8, 0, q, outs[0])

    def us(out):                                                        # the least of several, each of 30 launches
        ev = [torch.cuda.Event(enable_timing=True) for _ in range(9)]
        for e in ev:
            e.record()
            for _ in range(30):
                rig.kvd.step_layers(0, 8, 0, q, out)
        torch.cuda.synchronize()
        return min(a.elapsed_time(b) for a, b in zip(ev[1:], ev[2:])) / 30 * 1e3 / 8

    rule = us(outs[1])
    shape = rig.kvd.step_shape(multi_layer=True)
    assert shape[2] == 16
    rig.kvd.set_step_shape(*shape, multi_layer=True)
    again = us(outs[2])
    print(f"rule {rule:.2f} us a layer, set {again:.2f}")
    assert again < 1.2 * rule
    chosen, us_chosen, us_rule = rig.kvd.calibrate_step_shape(0, 0, q, outs[2], launches_per_shape=4, n_layers=8)
    kept = us(outs[2])
    rig.kvd.set_step_shape(*chosen, multi_layer=True)
    assert rig.kvd.step_shape(multi_layer=True) == chosen
    assert us(outs[2]) < 1.2 * kept
    rig.kvd.set_step_shape(multi_layer=True)
    rig.kvd.step_layers(0, 8, 0, q, outs[2])
    torch.cuda.synchronize()
    assert torch.equal(outs[1], outs[0]) and torch.equal(outs[2], outs[0])
    rig.close()
