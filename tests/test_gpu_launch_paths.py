"""GPU: the paths a plan and its tiles take to the device, at the sizes where they can go wrong."""
import numpy as np
import pytest

import synthetic_inputs as si
from gpu_helpers import from_dev_u16, gpu_step, to_dev_u16
from helpers import bits_to_f32, check_close, oracle_out, oracle_pool

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B", [1, 291, 292, 293, 585])
def test_plan_upload_around_its_workgroup_size(B):
    """A plan is copied 16 KiB to a workgroup: 56 B per tile put 292 tiles and the queue bounds at the first edge."""
    rng = np.random.default_rng(B)
    b = si.make_batch("upload", L=rng.integers(0, 40, B), n=np.ones(B, np.int32), Hq=2, Hkv=1, D=64, seed=B)
    _, out, stats = gpu_step(b)
    assert stats["n_items"] == B
    check_close(bits_to_f32(out), oracle_out(b))


def test_plans_follow_one_another_through_the_staging_buffers():
    """More plans than staging buffers, enqueued without a wait: each step must read its own."""
    import torch
    import paper_2603_13358_amd as ppd

    dev = torch.device("cuda:0")
    rng = np.random.default_rng(3)
    full = si.make_batch("plans", L=rng.integers(40, 300, 24), n=np.ones(24, np.int32), Hq=8, Hkv=2, D=64, seed=3)
    pool_bits = oracle_pool(full)
    ctx = ppd.Context(full.Hq, full.Hkv, full.D, full.num_pages)
    pool, pt = to_dev_u16(pool_bits, torch, dev), torch.from_numpy(full.page_tables).to(dev)
    steps, outs = [], []
    for k in range(11):  # every step sees another prefix of every sequence
        b = si.make_batch("plans", L=np.maximum(full.L - 3 * k, 0), n=full.n, Hq=8, Hkv=2, D=64, seed=50 + k,
                          page_tables=full.page_tables, num_pages=full.num_pages)
        steps.append(b)
        outs.append((to_dev_u16(b.q, torch, dev), torch.zeros((b.T, b.Hq, b.D), dtype=torch.int16, device=dev)))
    torch.cuda.synchronize()
    for b, (q, out) in zip(steps, outs):
        ctx.mixed_attention(q, pool, pt, b.L, b.n, b.scale, out)
    torch.cuda.synchronize()
    for b, (_, out) in zip(steps, outs):
        check_close(bits_to_f32(from_dev_u16(out).reshape(b.T, b.Hq, b.D)), oracle_out(b, pool_bits))
    ctx.close()
