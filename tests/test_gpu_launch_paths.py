"""GPU: the paths a plan and its tiles take to the device, at the sizes where they can go wrong."""
import numpy as np
import pytest

import oracle
import synthetic_inputs as si
from gpu_helpers import from_dev_u16, gpu_step, gpu_step_fp8, to_dev_u16
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


@pytest.mark.parametrize("static", [False, True])
def test_a_host_that_runs_ahead_waits_for_its_own_uploads_only(static):
    """More plans in flight than staging buffers (the entry point that allocates nothing has one), three layers each, while
    another stream is busy for long: the calls return before that stream is done, and every step has read its own plan."""
    import torch
    import paper_2603_13358_amd as ppd

    dev = torch.device("cuda:0")
    rng = np.random.default_rng(9)
    full = si.make_batch("ahead", L=rng.integers(40, 300, 24), n=np.ones(24, np.int32), Hq=8, Hkv=2, D=64, seed=9)
    pool_bits = oracle_pool(full)
    ctx = ppd.Context(full.Hq, full.Hkv, full.D, full.num_pages)
    pool, pt = to_dev_u16(pool_bits, torch, dev), torch.from_numpy(full.page_tables).to(dev)
    call = ctx.mixed_attention_static if static else ctx.mixed_attention
    steps = []
    for k in range(10):
        b = si.make_batch("ahead", L=np.maximum(full.L - 3 * k, 0), n=full.n, Hq=8, Hkv=2, D=64, seed=70 + k,
                          page_tables=full.page_tables, num_pages=full.num_pages)
        steps.append((b, to_dev_u16(b.q, torch, dev), torch.zeros((b.T, b.Hq, b.D), dtype=torch.int16, device=dev)))
    for k in range(5):  # every buffer has its size, every kernel has been loaded
        call(steps[k][1], pool, pt, steps[k][0].L, steps[k][0].n, steps[k][0].scale, steps[k][2])
    x = torch.randn(8192, 8192, device=dev, dtype=torch.bfloat16)
    y = torch.empty_like(x)
    torch.mm(x, x, out=y)
    torch.cuda.synchronize()
    other, busy = torch.cuda.Stream(), torch.cuda.Event()
    with torch.cuda.stream(other):
        for _ in range(400):
            torch.mm(x, x, out=y)
        busy.record()
    for b, q, out in steps:
        for _ in range(3):
            call(q, pool, pt, b.L, b.n, b.scale, out)
    assert not busy.query()
    torch.cuda.synchronize()
    for b, _, out in steps:
        check_close(bits_to_f32(from_dev_u16(out).reshape(b.T, b.Hq, b.D)), oracle_out(b, pool_bits))
    ctx.close()


@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("D,Hkv,T,layers", [(128, 8, 1023, 1), (128, 8, 1025, 1), (64, 8, 1021, 1), (64, 2, 1031, 4), (128, 1, 7, 1)])
def test_append_on_both_sides_of_its_token_split(D, Hkv, T, layers, fp8):
    """8 or 16 tokens per workgroup by T * Hkv * layers (the line is 8192): runs of every length from every offset, with
    skipped tokens, and a batch end inside a workgroup; every byte of the pools against the oracle."""
    import oracle
    import torch
    import paper_2603_13358_amd as ppd

    rng = np.random.default_rng(T + D)
    slots, page = [], 0
    while len(slots) < T:
        run, off = int(rng.integers(1, 60)), int(rng.integers(0, 16))
        s = page * 16 + off + np.arange(run)
        s[rng.random(run) < 0.03] = -1
        slots.extend(s.tolist())
        page += (off + run + 15) // 16
    slots = np.asarray(slots[:T], np.int64)
    num_pages = page + 1
    k, v = (si.normal_bf16(rng, (layers, T, Hkv, D)) for _ in range(2))
    per = oracle.pool_elems(num_pages, Hkv, D, 16)
    ref = np.full((layers, per), 0x5A, np.uint8 if fp8 else np.uint16)
    for i in range(layers):
        if fp8:
            oracle.kv_append_fp8(k[i], v[i], ref[i], slots, Hkv, D, 16, num_pages, 0.02, 0.05)
        else:
            oracle.kv_append(k[i], v[i], ref[i], slots, Hkv, D, 16, num_pages)
    dev = torch.device("cuda:0")
    ctx = ppd.Context(2 * Hkv, Hkv, D, num_pages)
    if fp8:
        ctx.set_kv_format(ppd.PPD_KV_FP8_E4M3, 0.02, 0.05)
    pools = torch.full((layers, per), 0x5A, dtype=torch.uint8 if fp8 else torch.int16, device=dev)
    ctx.kv_land(to_dev_u16(k, torch, dev), to_dev_u16(v, torch, dev), pools, per, layers, torch.from_numpy(slots).to(dev))
    torch.cuda.synchronize()
    assert ctx.device_error_flags() == 0
    got = pools.cpu().numpy()
    assert np.array_equal(got if fp8 else got.view(np.uint16), ref)
    ctx.close()


@pytest.mark.parametrize("D,chunk", [(128, 0), (128, 64), (64, 192)])
@pytest.mark.parametrize("q_std", [0.5, 6.0, 40.0])
def test_row_block_reference_is_raised_and_found(D, chunk, q_std):
    """Row-block tiles look for a maximum only when a sum of exponentials grows past a bound or no reference exists: flat
    scores (never after the first tile), scores that grow by far more than the bound, and splits of 64 keys on the causal
    edge, where some columns see no key of the split's first tile."""
    b = si.make_batch("reference", L=[1000, 0, 70, 333], n=[70, 300, 130, 61], Hq=8, Hkv=2, D=D, seed=int(q_std * 10) + D,
                      q_std=q_std, slack_pages=3)
    _, out, stats = gpu_step(b, options={"mfma_chunk": chunk} if chunk else None)
    assert stats["n_mfma"] > 0
    # peaky rows give back single values: bf16 rounds a probability and the result by at most 2^-8 of their size each
    check_close(bits_to_f32(out), oracle_out(b), max_abs=2.0 ** -7 * float(np.abs(bits_to_f32(b.v)).max()))


@pytest.mark.parametrize("bits_above", [7.0, 9.0, 12.0])
def test_row_block_probabilities_stay_below_their_bound(bits_above):
    """A key whose score lies `bits_above` powers of two over the running reference, with V of 1.5e35: a probability of more
    than 2^8 against an old reference would leave binary32 in the sum, although the result is an ordinary number."""
    b = si.make_batch("large_v", L=[200], n=[70], Hq=8, Hkv=1, D=128, seed=5)
    b.q[:] = 0
    b.q[..., 0] = 0x3F80
    b.k[:] = 0
    b.k[150, 0, :1] = si.f32_to_bf16_bits(np.array([bits_above * np.log(2.0) / b.scale]))
    rng = np.random.default_rng(5)
    b.v[:] = si.f32_to_bf16_bits(rng.choice([-1.0, 1.0], b.v.shape).astype(np.float32) * np.float32(1.5e35))
    _, out, stats = gpu_step(b)
    assert stats["n_mfma"] == 3 and stats["n_groups"] == 0
    check_close(bits_to_f32(out) / 1.5e35, oracle_out(b) / 1.5e35)


@pytest.mark.parametrize("Hq,Hkv,D", [(8, 8, 128), (10, 2, 128), (8, 1, 128), (6, 2, 64), (7, 1, 64)])
@pytest.mark.parametrize("fp8", [False, True])
def test_row_block_results_leave_whole_lines(Hq, Hkv, D, fp8):
    """A wave writes its 32 columns through LDS, half a row at a time: row blocks that end one column into a wave, at its
    edge and inside it, for group sizes that divide 32 and that do not; what surrounds the result stays as it was."""
    import torch
    import paper_2603_13358_amd as ppd

    G = Hq // Hkv
    n = [17, 32 // G + 1, 256 // G, 256 // G + 1, 2 * (256 // G) - 1, 33]
    n = [max(x, 16 // G + 1) for x in n]
    b = si.make_batch("lines", L=[5, 0, 100, 64, 31, 0], n=n, Hq=Hq, Hkv=Hkv, D=D, seed=Hq * D, slack_pages=3)
    dev = torch.device("cuda:0")
    ctx = ppd.Context(Hq, Hkv, D, b.num_pages)
    if fp8:
        ctx.set_kv_format(ppd.PPD_KV_FP8_E4M3, 0.0173, 0.0421)
        pool = torch.zeros(ctx.pool_elems(), dtype=torch.uint8, device=dev)
    else:
        pool = torch.zeros(ctx.pool_elems(), dtype=torch.int16, device=dev)
    for k, v, slots in (b.cached_part(), b.new_part()):
        ctx.kv_append(to_dev_u16(k, torch, dev), to_dev_u16(v, torch, dev), pool, torch.from_numpy(slots.astype(np.int64)).to(dev))
    rows = torch.full((b.T + 2, Hq, D), 0x7A5A, dtype=torch.int16, device=dev)
    ctx.mixed_attention(to_dev_u16(b.q, torch, dev), pool, torch.from_numpy(b.page_tables).to(dev), b.L, b.n, b.scale, rows[1:])
    torch.cuda.synchronize()
    assert ctx.device_error_flags() == 0 and ctx.plan_stats().as_dict()["n_mfma"] > 0
    got = from_dev_u16(rows)
    assert (got[0] == 0x7A5A).all() and (got[-1] == 0x7A5A).all()
    want = oracle_out(b)
    if fp8:  # the oracle reads the codes the append wrote
        want = oracle.mixed_attention_fp8(b.q, pool.cpu().numpy(), 0.0173, 0.0421, b.page_tables, b.L, b.n, Hq, Hkv, D, b.P,
                                          b.num_pages, b.scale)
    check_close(bits_to_f32(got[1:-1]), want)
    ctx.close()


@pytest.mark.parametrize("B_narrow,B_rows,wave", [(1, 1, -1), (3, 9, -1), (9, 2, -1), (30, 25, -1), (30, 25, 1), (31, 33, -1), (32, 33, -1)])
def test_mixed_launch_with_a_workgroup_for_every_tile(B_narrow, B_rows, wave):
    """Up to 256 tiles are taken by workgroup index (8 to 256 here), more (260) are claimed: row blocks in few and in all
    of the eight queues, one and several per sharing group, wave tiles, and the same call with one workgroup."""
    rng = np.random.default_rng(B_narrow * 100 + B_rows)
    L = np.concatenate([rng.integers(0, 500, B_narrow), rng.integers(0, 300, B_rows)])
    n = np.concatenate([np.ones(B_narrow, np.int64), rng.integers(17, 150, B_rows)])
    b = si.make_batch("own", L=L, n=n, Hq=4, Hkv=4, D=64, seed=B_rows, slack_pages=3)
    _, out, stats = gpu_step(b, options={"wave_tiles": wave})
    assert stats["n_mfma"] == 4 * B_rows and stats["n_narrow"] == 4 * B_narrow
    check_close(bits_to_f32(out), oracle_out(b))
    _, claimed, _ = gpu_step(b, options={"wave_tiles": wave, "grid": 1})
    assert np.array_equal(out, claimed)


@pytest.mark.parametrize("fp8,longest", [(False, 768), (True, 1536)])
def test_decode_only_launch_of_many_short_tiles(fp8, longest):
    """2048 decode tiles, most of them of at most 300 keys (which run one per wave), a few of up to 768 or 1536 (which do
    not), whole and partly filled last pages among them."""
    import torch  # noqa: F401 -- before the library: both load a HIP runtime, and torch has to find its own
    import paper_2603_13358_amd as ppd

    rng = np.random.default_rng(longest)
    L = rng.integers(0, 300, 256)
    L[:6] = [longest - 1, longest - 2, longest - 16, longest - 17, 15, 16]
    items, _ = ppd.ppd_plan_build(8, 8, 128, 16, 1 << 20, L, np.ones(256, np.int64))
    assert sorted({t.queue for t in items}) == [8, 9] and sum(t.queue == 9 for t in items) == 8 * 252
    b = si.make_batch("single", L=L, n=np.ones(256, np.int64), Hq=8, Hkv=8, D=128, seed=longest, slack_pages=3)
    if fp8:
        pool, out, _ = gpu_step_fp8(b, 0.0173, 0.0421)
        want = oracle.mixed_attention_fp8(b.q, pool, 0.0173, 0.0421, b.page_tables, b.L, b.n, b.Hq, b.Hkv, b.D, b.P, b.num_pages, b.scale)
    else:
        _, out, _ = gpu_step(b)
        want = oracle_out(b)
    check_close(bits_to_f32(out), want)


@pytest.mark.parametrize("Hq,Hkv,D", [(16, 8, 128), (16, 8, 64)])
@pytest.mark.parametrize("fp8", [False, True])
def test_short_decode_batch_is_as_exact_as_on_whole_workgroups(Hq, Hkv, D, fp8):
    """256 sequences of 64-700 keys: the tiles that the planner chooses have no more error than tiles that all run on eight
    waves.  Both errors are means over 2^18 and more results, which one tile kind repeats to within 0.3 % over seeds."""
    rng = np.random.default_rng(D)
    b = si.make_batch("exact", L=rng.integers(64, 701, 256), n=np.ones(256, np.int64), Hq=Hq, Hkv=Hkv, D=D, seed=D, slack_pages=3)
    errors = []
    for options in ({}, {"wave_tiles": 0}):
        if fp8:
            pool, out, _ = gpu_step_fp8(b, 0.0173, 0.0421, options=options)
            want = oracle.mixed_attention_fp8(b.q, pool, 0.0173, 0.0421, b.page_tables, b.L, b.n, Hq, Hkv, D, b.P, b.num_pages, b.scale)
        else:
            _, out, _ = gpu_step(b, options=options)
            want = oracle_out(b)
        d = bits_to_f32(out).astype(np.float64) - want
        errors.append(np.sqrt((d * d).sum() / (np.asarray(want, np.float64) ** 2).sum()))
    assert errors[0] <= 1.01 * errors[1], errors


@pytest.mark.parametrize("D,G,L", [(128, 4, [1534] * 3), (128, 4, [1535] * 3), (128, 8, [3000, 61, 47, 3049]), (128, 1, [0, 15, 16, 6000]),
                                   (64, 4, [1535, 4000, 1])])
def test_decode_only_kernel_for_short_and_for_long_tiles(D, G, L):
    """Tiles of 1535, of 1536 and of mixed lengths on average (the decode-only kernel takes other register sets from 1536
    on): the oracle's result, and bit for bit the mixed kernel's."""
    b = si.make_batch("sets", L=L, n=np.ones(len(L), np.int64), Hq=8 * G, Hkv=8, D=D, seed=D + G + len(L), slack_pages=2)
    options = {"narrow_chunk": 8192}
    _, out, stats = gpu_step(b, options=options)
    assert stats["n_narrow"] == 8 * len(L)
    check_close(bits_to_f32(out), oracle_out(b))
    _, mixed, _ = gpu_step(b, options=dict(options, narrow_kernel=0))
    assert np.array_equal(out, mixed)


@pytest.mark.parametrize("Hq,Hkv,D,L,n,chunk", [
    (32, 8, 128, [900, 17, 4000, 0, 2047], [1, 1, 1, 4, 1], 256),   # 1..16 splits, whole ranges beside them
    (8, 8, 128, [8191], [1], 64),                                   # one column, 128 splits
    (16, 2, 64, [3000, 129], [2, 1], 64),                           # 16 columns: two passes of the merging workgroup
    (40, 8, 128, [577, 511, 512], [3, 1, 1], 64),                   # 15 and 5 columns
    (16, 2, 128, [17000], [2], 64),                                 # 16 columns x 266 splits: more pairs than are staged
])
@pytest.mark.parametrize("fp8", [False, True])
def test_split_ranges_are_merged_by_their_last_tile(Hq, Hkv, D, L, n, chunk, fp8):
    """Decode-only launches of one round merge split ranges themselves: the oracle's result, bit for bit that of the mixed
    kernel and the merge launch behind it, and again on the same plan (the counts are back at zero)."""
    import torch
    import paper_2603_13358_amd as ppd

    b = si.make_batch("last", L=L, n=n, Hq=Hq, Hkv=Hkv, D=D, seed=D + len(L), slack_pages=2)
    options = {"narrow_chunk": chunk, "grid": 1 << 12}  # a workgroup for every tile
    if fp8:
        pool, out, stats = gpu_step_fp8(b, 0.0173, 0.0421, options=options)
        want = oracle.mixed_attention_fp8(b.q, pool, 0.0173, 0.0421, b.page_tables, b.L, b.n, Hq, Hkv, D, b.P, b.num_pages, b.scale)
        _, mixed, _ = gpu_step_fp8(b, 0.0173, 0.0421, options=dict(options, narrow_kernel=0))
    else:
        pool, out, stats = gpu_step(b, options=options)
        want = oracle_out(b)
        _, mixed, _ = gpu_step(b, options=dict(options, narrow_kernel=0))
    assert stats["n_groups"] > 0 and stats["n_mfma"] == 0 and stats["n_items"] <= stats["grid"]
    check_close(bits_to_f32(out), want)
    assert np.array_equal(out, mixed)
    dev = torch.device("cuda:0")
    ctx = ppd.Context(Hq, Hkv, D, b.num_pages)
    if fp8:
        ctx.set_kv_format(ppd.PPD_KV_FP8_E4M3, 0.0173, 0.0421)
    for key, value in options.items():
        ctx.set_option(key, value)
    dpool = torch.from_numpy(pool if fp8 else pool.view(np.int16)).to(dev)
    q, pt = to_dev_u16(b.q, torch, dev), torch.from_numpy(b.page_tables).to(dev)
    for call in (ctx.mixed_attention, ctx.mixed_attention, ctx.mixed_attention_static, ctx.mixed_attention_static):
        got = torch.zeros((b.T, b.Hq, b.D), dtype=torch.int16, device=dev)
        call(q, dpool, pt, b.L, b.n, b.scale, got)
        torch.cuda.synchronize()
        assert np.array_equal(from_dev_u16(got).reshape(out.shape), out)
    ctx.close()


@pytest.mark.parametrize("G,rows,chunk", [(4, 1, 8192), (1, 16, 8192), (8, 2, 8192), (5, 3, 4096)])
def test_rounds_of_long_tiles_run_on_four_waves(G, rows, chunk):
    """Decode-only launches of at least two rounds of tiles of 3072 keys and more (64 sequences that share two sequences' pages, 8 KV
    heads; with split ranges in the last case): the oracle's result, with less error than eight waves have, whose probabilities
    are rounded once (0.71 of it was measured)."""
    import torch
    import paper_2603_13358_amd as ppd

    B, longest = 64, 8192 if chunk < 8192 else 4400
    rng = np.random.default_rng(G)
    base = si.make_batch("four", L=[longest - 1, longest - 9], n=[1, 1], Hq=8, Hkv=8, D=128, seed=G, slack_pages=2)
    pool, _, _ = gpu_step(base)
    low = 6400 if chunk < 8192 else 3100
    n = np.where(np.arange(B) % 5 == 0, rows, 1).astype(np.int32)
    L = (rng.integers(low, longest - 30, B)).astype(np.int32)
    L[:4] = [low, longest - 30, (longest - 30) // 16 * 16 - 1, (longest - 30) // 16 * 16]
    tables = base.page_tables[np.arange(B) % 2]
    q = (rng.standard_normal((int(n.sum()), 8 * G, 128)).astype(np.float32).view(np.uint32) >> 16).astype(np.uint16)
    scale = 1.0 / np.sqrt(128.0)
    want = oracle.mixed_attention(q, pool, tables, L, n, 8 * G, 8, 128, 16, base.num_pages, scale)
    dev = torch.device("cuda:0")
    dpool, dq, dt = to_dev_u16(pool, torch, dev), to_dev_u16(q, torch, dev), torch.from_numpy(np.ascontiguousarray(tables)).to(dev)
    errors = []
    for narrow_kernel in (1, 0):
        ctx = ppd.Context(8 * G, 8, 128, base.num_pages)
        ctx.set_option("narrow_chunk", chunk)
        ctx.set_option("narrow_kernel", narrow_kernel)
        out = torch.zeros((len(q), 8 * G, 128), dtype=torch.int16, device=dev)
        ctx.mixed_attention(dq, dpool, dt, L, n, scale, out)
        torch.cuda.synchronize()
        stats = ctx.plan_stats()
        assert stats.n_mfma == 0 and stats.n_narrow >= 512 and stats.kv_bytes_tiles >= stats.n_narrow * 512 * 3072
        assert (stats.n_groups > 0) == (chunk < 8192) and ctx.device_error_flags() == 0
        got = bits_to_f32(from_dev_u16(out)).reshape(want.shape)
        check_close(got, want)
        errors.append(np.linalg.norm(got.astype(np.float64) - want))
        ctx.close()
    assert errors[0] <= 0.875 * errors[1], errors


@pytest.mark.parametrize("B", [8, 9, 15, 16, 17, 25])
@pytest.mark.parametrize("fp8,wave", [(False, 0), (True, 0), (False, 1)])
def test_two_rounds_of_short_tiles_are_handed_out_by_index(B, fp8, wave):
    """Around one and two slots for each of 8 workgroups (from the 17th on they are claimed): the oracle's result, bit for bit the
    mixed kernel's, twice."""
    rng = np.random.default_rng(B)
    L = rng.integers(0, 900, B)
    L[:2] = [1535, 0]
    b = si.make_batch("index", L=L, n=np.ones(B, np.int64), Hq=4, Hkv=1, D=128, seed=B, slack_pages=2)
    options = {"grid": 8, "wave_tiles": wave, "narrow_chunk": 2048}

    def step(extra):
        if fp8:
            return gpu_step_fp8(b, 0.0173, 0.0421, options=dict(options, **extra))
        return gpu_step(b, options=dict(options, **extra))

    pool, out, stats = step({})
    assert stats["n_items"] == B
    want = oracle.mixed_attention_fp8(b.q, pool, 0.0173, 0.0421, b.page_tables, b.L, b.n, 4, 1, 128, b.P, b.num_pages, b.scale) if fp8 else oracle_out(b)
    check_close(bits_to_f32(out), want)
    for extra in ({}, {"narrow_kernel": 0}):
        assert np.array_equal(step(extra)[1], out)


@pytest.mark.parametrize("static", [False, True])
@pytest.mark.parametrize("G,grid", [(4, 0), (4, 1024), (1, 720), (8, 512)])
def test_long_split_tiles_are_merged_whatever_the_grid(G, grid, static):
    """Decode-only launches of at least two rounds of long tiles with split ranges, whole ones and ranges of one to three
    pages beside them, with fewer workgroups than tiles (grid 0) and with one for each (the sequences share two sequences'
    pages): the oracle's result, bit for bit that of the automatic grid."""
    import torch
    import paper_2603_13358_amd as ppd

    B, longest = 48, 13000
    rng = np.random.default_rng(G)
    base = si.make_batch("grid", L=[longest - 1, longest - 9], n=[1, 1], Hq=8, Hkv=8, D=128, seed=G, slack_pages=2)
    pool, _, _ = gpu_step(base)
    L = rng.integers(8200, longest - 30, B).astype(np.int32)
    L[:8] = [0, 15, 40, 47, 5000, 8191, 8192, longest - 30]
    n = np.ones(B, np.int32)
    tables = np.ascontiguousarray(base.page_tables[np.arange(B) % 2])
    q = (rng.standard_normal((B, 8 * G, 128)).astype(np.float32).view(np.uint32) >> 16).astype(np.uint16)
    scale = 1.0 / np.sqrt(128.0)
    want = oracle.mixed_attention(q, pool, tables, L, n, 8 * G, 8, 128, 16, base.num_pages, scale)
    dev = torch.device("cuda:0")
    dpool, dq, dt = to_dev_u16(pool, torch, dev), to_dev_u16(q, torch, dev), torch.from_numpy(tables).to(dev)
    outs = []
    for g in (grid, 0):
        ctx = ppd.Context(8 * G, 8, 128, base.num_pages)
        ctx.set_option("narrow_chunk", 8192)
        ctx.set_option("grid", g)
        call = ctx.mixed_attention_static if static else ctx.mixed_attention
        for _ in range(2):
            out = torch.zeros((B, 8 * G, 128), dtype=torch.int16, device=dev)
            call(dq, dpool, dt, L, n, scale, out)
            torch.cuda.synchronize()
            outs.append(from_dev_u16(out))
        stats = ctx.plan_stats()
        assert stats.n_mfma == 0 and stats.n_groups > 0 and stats.n_items == 720 and ctx.device_error_flags() == 0  # 2.8 rounds
        assert stats.kv_bytes_tiles >= stats.n_items * 512 * 3072 and (g == 0 or stats.n_items <= stats.grid or g == 512)
        ctx.close()
    check_close(bits_to_f32(outs[0]).reshape(want.shape), want)
    for other in outs[1:]:
        assert np.array_equal(outs[0], other)


@pytest.mark.parametrize("options", [{}, {"narrow_chunk": 4096}])
def test_infinite_values_stay_infinite_on_four_waves(options):
    """Decode-only launches of at least two rounds of long tiles over V elements of +inf and of -inf, of one key and of
    several (the keys of a wave's largest probability among them): those columns of every row that sees them are infinite, as
    they are on eight waves, and the other columns do not notice."""
    import torch
    import paper_2603_13358_amd as ppd

    B, Hq, D, longest = 64, 16, 128, 8192
    rng = np.random.default_rng(7)
    base = si.make_batch("inf", L=[longest - 1] * 2, n=[1, 1], Hq=8, Hkv=8, D=D, seed=7, slack_pages=2)
    pool, _, _ = gpu_step(base)
    finite = pool.copy()
    v = pool.reshape(base.num_pages, 2, 8, 2, D, 8)[:, 1]  # page, head, token octet, d, token of the octet (a view)
    columns = np.arange(0, D, 3)
    sign = np.where(columns % 2, -1.0, 1.0)
    for s in range(2):
        for i, d in enumerate(columns):
            # one key for some columns, every key of the first 4096 for others
            keys = rng.integers(0, 4096, 1) if i % 3 else np.arange(4096)
            v[base.page_tables[s, keys // 16], :, keys % 16 // 8, d, keys % 8] = 0x7F80 if sign[i] > 0 else 0xFF80
    L = rng.integers(6200, longest - 30, B).astype(np.int32)
    n = np.ones(B, np.int32)
    tables = np.ascontiguousarray(base.page_tables[np.arange(B) % 2])
    q = (rng.standard_normal((B, Hq, D)).astype(np.float32).view(np.uint32) >> 16).astype(np.uint16)
    scale = 1.0 / np.sqrt(D)
    dev = torch.device("cuda:0")
    dq, dt = to_dev_u16(q, torch, dev), torch.from_numpy(tables).to(dev)

    def run(bits, narrow_kernel):
        ctx = ppd.Context(Hq, 8, D, base.num_pages)
        for key, value in dict({"narrow_chunk": 8192}, **options).items():
            ctx.set_option(key, value)
        ctx.set_option("narrow_kernel", narrow_kernel)
        out = torch.zeros((B, Hq, D), dtype=torch.int16, device=dev)
        ctx.mixed_attention(dq, to_dev_u16(bits, torch, dev), dt, L, n, scale, out)
        torch.cuda.synchronize()
        stats = ctx.plan_stats()
        assert stats.n_mfma == 0 and stats.n_items >= 512 and stats.kv_bytes_tiles >= stats.n_items * 512 * 3072
        ctx.close()
        return bits_to_f32(from_dev_u16(out)).reshape(B, Hq, D)

    plain = run(finite, 1)
    for narrow_kernel in (0, 1):
        got = run(pool, narrow_kernel)
        assert np.array_equal(got[:, :, columns], np.broadcast_to(sign * np.inf, (B, Hq, len(columns)))), narrow_kernel
        rest = np.setdiff1d(np.arange(D), columns)
        if narrow_kernel:
            assert np.array_equal(got[:, :, rest], plain[:, :, rest])


@pytest.mark.parametrize("L,options", [([510] * 5, {}), ([511] * 5, {}), ([5000, 3, 47, 801], {}), ([200] * 40 + [3000], {}),
                                       ([9000, 31, 2500], {"narrow_chunk": 960}), ([9000, 31, 2500], {"narrow_chunk": 1024}),
                                       ([300] * 17 + [12], {"wave_tiles": 1}), ([380] * 9 + [4000] * 3, {"wave_tiles": 1})])
def test_decode_only_kernel_on_fp8_pages_of_head_size_64(L, options):
    """Tiles of 511, of 512 and of mixed lengths (the decode-only kernel takes other register sets from 512 on, 1024 where it
    merges), split and on single waves: the oracle's result, and bit for bit the mixed kernel's."""
    b = si.make_batch("sets8", L=L, n=np.ones(len(L), np.int64), Hq=32, Hkv=8, D=64, seed=len(L), slack_pages=2)
    options = dict({"narrow_chunk": 8192}, **options)
    pool, out, stats = gpu_step_fp8(b, 0.0173, 0.0421, options=options)
    assert stats["n_mfma"] == 0
    check_close(bits_to_f32(out), oracle.mixed_attention_fp8(b.q, pool, 0.0173, 0.0421, b.page_tables, b.L, b.n, 32, 8, 64, b.P, b.num_pages, b.scale))
    _, mixed, _ = gpu_step_fp8(b, 0.0173, 0.0421, options=dict(options, narrow_kernel=0))
    assert np.array_equal(out, mixed)


@pytest.mark.parametrize("B,Hkv,D,n_long,options", [(80, 8, 128, 0, {}), (83, 8, 64, 0, {"grid": 7}), (161, 4, 128, 0, {}),
                                                    (200, 8, 128, 25, {"grid": 4096}), (230, 7, 64, 30, {}), (256, 8, 128, 251, {}),
                                                    (520, 8, 64, 500, {}), (40, 8, 128, 0, {}), (67, 8, 64, 0, {"grid": 300})])
@pytest.mark.parametrize("fp8", [False, True])
def test_decode_tiles_on_single_waves(B, Hkv, D, n_long, options, fp8):
    """Launches of 640 short tiles and more (FP8 pages: of more than 256), a wave to a tile: pages, and units of tiles, that are not full, one to three rounds of
    the waves, multi-row tiles, infinite V.  The oracle's result, the same whatever the grid, and with less error than on whole
    workgroups (one bf16 rounding less: 0.71 of it where the results are averages over many keys)."""
    rng = np.random.default_rng(B + D)
    L = rng.integers(70, 140, B) if B * Hkv >= 640 else rng.integers(60, 90, B)
    L[B - n_long:] = rng.integers(384, 420, n_long)
    L[1:5] = [0, 15, 16, 17]
    n = np.where(np.arange(B) % 9 == 8, 2, 1)
    b = si.make_batch("waves", L=L, n=n, Hq=4 * Hkv, Hkv=Hkv, D=D, seed=B, slack_pages=3)
    b.v[5] = 0x7F80  # positive infinity (bf16), in the first sequence: every result there (the largest code on FP8 pages)
    errors, outs = [], []
    for extra in ({}, {"grid": 0}, {"wave_tiles": 0, "grid": 0}):
        if fp8:
            pool, out, stats = gpu_step_fp8(b, 0.0173, 0.0421, options=dict(options, **extra))
            want = oracle.mixed_attention_fp8(b.q, pool, 0.0173, 0.0421, b.page_tables, b.L, b.n, b.Hq, b.Hkv, b.D, b.P, b.num_pages, b.scale)
        else:
            _, out, stats = gpu_step(b, options=dict(options, **extra))
            want = oracle_out(b)
        assert stats["n_narrow"] > 256 and stats["n_mfma"] == 0
        got, finite = bits_to_f32(out), np.isfinite(want)
        assert np.array_equal(got[~finite], want[~finite]) and finite[1:].all() and finite[0].any() == fp8
        check_close(got[1:], want[1:])
        errors.append(np.linalg.norm(got[5:].astype(np.float64) - want[5:]))
        outs.append(out)
    assert np.array_equal(outs[0], outs[1])
    assert errors[0] <= (0.875 if fp8 or B * Hkv >= 640 else 1) * errors[2], errors


@pytest.mark.parametrize("B,Hkv,D,grid,rows", [(33, 8, 128, 0, 2), (80, 8, 128, 0, 3), (37, 2, 128, 8, 3), (49, 1, 128, 16, 3), (48, 1, 64, 16, 3), (23, 3, 64, 5, 3), (130, 1, 128, 3, 3)])
def test_rounds_of_short_tiles_run_pipelined(B, Hkv, D, grid, rows):
    """Decode-only launches of 1.03 to 43 rounds of short whole-workgroup tiles on bf16 pages: three rounds go by index and the rest is
    claimed; shares of no page and of several, last pages partly filled, multi-row tiles.  The oracle's result, bit for bit the
    mixed kernel's, and again on one context (the cursor is left re-armed)."""
    import torch
    import paper_2603_13358_amd as ppd

    rng = np.random.default_rng(B)
    L = rng.integers(60, 420, B)
    L[:5] = [0, 15, 16, 17, 419]
    n = np.where(np.arange(B) % 7 == 6, rows, 1)
    b = si.make_batch("pipe", L=L, n=n, Hq=4 * Hkv, Hkv=Hkv, D=D, seed=B, slack_pages=3)
    options = {"grid": grid, "wave_tiles": 0}
    pool, out, stats = gpu_step(b, options=options)
    assert stats["n_mfma"] == 0 and stats["n_narrow"] == B * Hkv > stats["grid"] and stats["n_groups"] == 0
    check_close(bits_to_f32(out), oracle_out(b))
    _, mixed, _ = gpu_step(b, options=dict(options, narrow_kernel=0))
    assert np.array_equal(out, mixed)
    dev = torch.device("cuda:0")
    ctx = ppd.Context(4 * Hkv, Hkv, D, b.num_pages)
    for key, value in options.items():
        ctx.set_option(key, value)
    dpool, q, pt = to_dev_u16(pool, torch, dev), to_dev_u16(b.q, torch, dev), torch.from_numpy(b.page_tables).to(dev)
    for call in (ctx.mixed_attention, ctx.mixed_attention, ctx.mixed_attention_static, ctx.mixed_attention):
        got = torch.zeros((b.T, b.Hq, b.D), dtype=torch.int16, device=dev)
        call(q, dpool, pt, b.L, b.n, b.scale, got)
        torch.cuda.synchronize()
        assert np.array_equal(from_dev_u16(got).reshape(out.shape), out)
    ctx.close()


@pytest.mark.parametrize("B,D,G,options,groups", [(34, 128, 4, {}, 176), (40, 64, 4, {"narrow_chunk": 256, "grid": 48}, 320), (37, 128, 8, {"narrow_chunk": 256, "grid": 100}, 296)])
def test_pipelined_tiles_of_split_ranges(B, D, G, options, groups):
    """Split ranges in pipelined launches, by the automatic split size and by a given one, in two rounds and in more: tiles that begin
    and end inside their sequence, whole ones beside them, multi-row tiles, partials that stay in the L2 and (more than 3 MiB) that do not.  The oracle's result, bit for bit the mixed kernel's, and
    again on one context, its static entry point among them."""
    import torch
    import paper_2603_13358_amd as ppd

    keys = 300 + np.arange(B) * 389 % 700  # tests/native/launch_forms_host.cpp, pipelined(): these launches are pipelined ones
    n = np.where(np.arange(B) % 7 == 6, 8 // G, 1)
    b = si.make_batch("split", L=keys - n, n=n, Hq=8 * G, Hkv=8, D=D, seed=B, slack_pages=3)
    pool, out, stats = gpu_step(b, options=options)
    assert stats["n_mfma"] == 0 and stats["n_narrow"] > stats["grid"] and stats["n_groups"] == groups
    assert (stats["partial_floats"] * 4 >= 3 << 20) == (G == 8)
    check_close(bits_to_f32(out), oracle_out(b))
    _, mixed, _ = gpu_step(b, options=dict(options, narrow_kernel=0))
    assert np.array_equal(out, mixed)
    dev = torch.device("cuda:0")
    ctx = ppd.Context(8 * G, 8, D, b.num_pages)
    for key, value in options.items():
        ctx.set_option(key, value)
    dpool, q, pt = to_dev_u16(pool, torch, dev), to_dev_u16(b.q, torch, dev), torch.from_numpy(b.page_tables).to(dev)
    for call in (ctx.mixed_attention, ctx.mixed_attention, ctx.mixed_attention_static, ctx.mixed_attention):
        got = torch.zeros((b.T, b.Hq, D), dtype=torch.int16, device=dev)
        call(q, dpool, pt, b.L, b.n, b.scale, got)
        torch.cuda.synchronize()
        assert np.array_equal(from_dev_u16(got).reshape(out.shape), out)
    ctx.close()


@pytest.mark.parametrize("fp8,D,B,low,high", [(False, 64, 256, 900, 1100), (False, 64, 200, 900, 1100), (True, 128, 128, 1900, 2100), (True, 64, 256, 1900, 2100)])
def test_long_decode_tiles_on_single_waves(fp8, D, B, low, high):
    """Tiles of more pages than a wave holds page ids of, around 64 and 128 pages, each on one wave (sequences that share two sequences'
    pages, 8 KV heads, every seventh with two rows): the oracle's result, with less error than on whole workgroups, as short tiles."""
    import torch
    import paper_2603_13358_amd as ppd

    Hq, Hkv = 16, 8
    rng = np.random.default_rng(B + D)
    keys = low + np.arange(B) * 37 % (high - low + 1)  # launch_forms_host.cpp, on_waves(): these launches run on single waves
    ends = [e for e in (2049, 2048, 2047, 2046, 1025, 1024, 1023, 1022, 15, 1) if e <= high]
    keys[:len(ends)] = ends
    n = np.where((np.arange(B) % 7 == 6) & (keys > 1), 2, 1).astype(np.int32)
    L = (keys - n).astype(np.int32)
    base = si.make_batch("long", L=[high, high], n=[1, 1], Hq=8, Hkv=Hkv, D=D, seed=B, slack_pages=2)
    tables = np.ascontiguousarray(base.page_tables[np.arange(B) % 2])
    q = (rng.standard_normal((int(n.sum()), Hq, D)).astype(np.float32).view(np.uint32) >> 16).astype(np.uint16)
    scale = 1.0 / np.sqrt(D)
    # The results over 15 and 1 keys are 10 to 40 times as large as those over 1000 and more, so the rounding of a few of them to bf16, which
    # both forms share, would outweigh what the forms differ by in all the others.
    averages = np.repeat(keys > 15, n)
    dev = torch.device("cuda:0")
    if fp8:
        pool, _, _ = gpu_step_fp8(base, 0.0173, 0.0421)
        want = oracle.mixed_attention_fp8(q, pool, 0.0173, 0.0421, tables, L, n, Hq, Hkv, D, 16, base.num_pages, scale)
        dpool = torch.from_numpy(pool).to(dev)
    else:
        pool, _, _ = gpu_step(base)
        want = oracle.mixed_attention(q, pool, tables, L, n, Hq, Hkv, D, 16, base.num_pages, scale)
        dpool = to_dev_u16(pool, torch, dev)
    dq, dt = to_dev_u16(q, torch, dev), torch.from_numpy(tables).to(dev)
    errors = []
    for wave_tiles in (-1, 0):
        ctx = ppd.Context(Hq, Hkv, D, base.num_pages)
        if fp8:
            ctx.set_kv_format(ppd.PPD_KV_FP8_E4M3, 0.0173, 0.0421)
        ctx.set_option("wave_tiles", wave_tiles)
        outs = []
        for _ in range(2):
            out = torch.zeros((len(q), Hq, D), dtype=torch.int16, device=dev)
            ctx.mixed_attention(dq, dpool, dt, L, n, scale, out)
            torch.cuda.synchronize()
            outs.append(from_dev_u16(out))
        stats = ctx.plan_stats()
        assert stats.n_narrow == B * Hkv and stats.n_mfma == 0 and stats.n_groups == 0 and ctx.device_error_flags() == 0
        assert np.array_equal(outs[0], outs[1])
        got = bits_to_f32(outs[0]).reshape(want.shape)
        check_close(got, want)
        errors.append(np.linalg.norm((got.astype(np.float64) - want)[averages]))
        ctx.close()
    assert errors[0] <= 0.875 * errors[1], errors
