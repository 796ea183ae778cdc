"""The result of a step does not depend on how a launch cuts its tiles up or on the order in which it takes them: drawn
tickets, every workgroup's own, and launches of a tensor each give the same bits.  (The tests' names are older than the half
and quarter tiles that launches consist of now.)"""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

# 25,394 tiles in halves; by themselves the four large tensors are launches of halves too, of another number of workgroups and
# tickets, the two small ones of quarters (test_gpu_units.py compares halves with quarters).  Ragged ends in the first, second
# and last quarter of a tile, one tensor of whole tiles only.
SIZES = [2048 * 6348 + 1, 2048 * 6349 - 900, 2048 * 6347, 2048 * 6348 + 777, 5, 2047]
PLANS = {"in_place": [(3, 5), (7, 8), (2, 6), (8, 4), (5, 3), (6, 7)],
         "transition": [(5, 3), (8, 7), (6, 2), (4, 5), (3, 3), (7, 6)],
         "wide": [(16, 5), (3, 32), (32, 16), (8, 16), (5, 32), (16, 7)]}


@pytest.fixture(scope="module")
def ctx():
    import paper_2604_06836_amd as stq
    c = stq.Context(0, 5000)
    yield c
    c.close()


def model(ctx, sizes, plan, K, seed, dtype="bf16"):
    from workloads import configs
    from workloads.harness import DeviceModel
    w = configs.Workload(seed, "schedules", [("t%d" % i, n) for i, n in enumerate(sizes)], K, dtype, 2, "normal_per_tensor")
    m = DeviceModel(ctx, w, plan, spare_width=32)
    return m


def launch(ctx, m, t, which, new=None, stats=False):
    """One step of the tensors `which` (indices) of the model; new: plan to write, into the spare buffers."""
    from paper_2604_06836_amd import binding
    from workloads.harness import hparams
    sub = (binding.Tensor * len(which))(*[m.tensors[l] for l in which])
    plan = binding.make_plan([m.plan[l] for l in which])
    hp = hparams(m.w, t, stats)
    if new is None:
        ctx.step(sub, plan, hp, m.stream)
    else:
        dst = [tuple(m._spare[(l, s)].data_ptr() if new[l][s] != m.plan[l][s] else None for s in (0, 1)) for l in which]
        ctx.step_transition(sub, plan, binding.make_plan([new[l] for l in which]), dst, hp, m.stream)


def outputs(m):
    torch.cuda.synchronize()
    return [[t.clone() for t in lst] for lst in (m.param, m.m_scales, m.v_scales, m.m_codes, m.v_codes)] + \
        [[m._spare[(l, s)].clone() for l in range(len(m.param)) for s in (0, 1)]]


@pytest.mark.parametrize("kind,dtype,tickets", [("in_place", "bf16", False), ("transition", "bf16", False)] +
                         [(kind, dtype, True) for kind in ("in_place", "transition", "wide") for dtype in ("bf16", "fp32")])
@pytest.mark.parametrize("stats", [False, True, "grad"])
def test_whole_tiles_and_quarters_give_the_same_bits(ctx, kind, dtype, tickets, stats):
    K = {"in_place": 64, "transition": 128, "wide": 256}[kind]
    got, sums = [], []
    for together in (False, True):
        plan = PLANS["in_place"] if kind == "transition" else PLANS[kind]
        new = PLANS["transition"] if kind == "transition" else None
        m = model(ctx, SIZES, plan, K, 70, dtype)
        for lst in (m.m_codes, m.v_codes):  # nothing undefined behind a state narrower than its buffer
            for l, buf in enumerate(lst):
                buf[m._code_words(SIZES[l], plan[l][0 if lst is m.m_codes else 1]):] = 0
        for s in m._spare.values():
            s.zero_()
        ctx.set_schedule(1 if together and tickets else 2 ** 63)
        m.set_grads(1)
        for t in (1, 2):
            which = [list(range(len(SIZES)))] if together else [[l] for l in range(len(SIZES))]
            for g in which:
                launch(ctx, m, t, g, new, stats)
                if stats and not together:
                    s = ctx.stats(1, m.stream)[0]
                    sums.append((t, g[0], [getattr(s, f) for f, _ in s._fields_]))
            if stats and together:
                for l, s in enumerate(ctx.stats(len(SIZES), m.stream)):
                    ref = dict(((a, b), c) for a, b, c in sums)[(t, l)]
                    for (f, _), a, b in zip(s._fields_, [getattr(s, f) for f, _ in s._fields_], ref):
                        if f == "count" or f.endswith("absmax"):
                            assert a == b, (l, f)
                        elif f == "g_sum":   # fp64 in another order: n * 2^-53 of the sum of absolute values
                            assert abs(a - b) <= 1e-12 * ref[2], (l, f)
                        elif f == "m_sum":   # of sqrt(n * sum of squares) >= the sum of absolute values (closer in test_gpu_units.py)
                            assert abs(a - b) <= 1e-5 * np.sqrt(SIZES[l] * ref[6]), (l, f)
                        else:
                            assert abs(a - b) <= (1e-12 if f.startswith("g_") else 1e-5) * abs(b) + SIZES[l] * 1.2e-38, (l, f)
        got.append(outputs(m))
        ctx.set_schedule(0)
        del m
    for a, b in zip(*got):
        for l, (x, y) in enumerate(zip(a, b)):
            assert torch.equal(x.view(torch.int32), y.view(torch.int32)), l


def test_tensor_search_over_three_levels(ctx):
    """4,700 small tensors in one launch (the search for a tile's tensor takes three rounds) against launches of 60."""
    sizes = [1 + (i * 7919) % 2500 for i in range(4700)]
    plan = [(2 + i % 7, 2 + (i // 7) % 7) for i in range(len(sizes))]
    got = []
    for group in (60, len(sizes)):
        m = model(ctx, sizes, plan, 64, 71)
        m.set_grads(1)
        for a in range(0, len(sizes), group):
            launch(ctx, m, 1, list(range(a, min(a + group, len(sizes)))))
        torch.cuda.synchronize()
        nm = [m._code_words(n, b) for n, (b, _) in zip(sizes, plan)]
        nv = [m._code_words(n, b) for n, (_, b) in zip(sizes, plan)]
        got.append([torch.cat(m.param).view(torch.int32), torch.cat(m.m_scales).view(torch.int32),
                    torch.cat([c[:k] for c, k in zip(m.m_codes, nm)]), torch.cat([c[:k] for c, k in zip(m.v_codes, nv)])])
        del m
    for x, y in zip(*got):
        assert torch.equal(x, y)


MANY = {  # (sizes, tensors per launch of the reference: its waves never skip, or walk)
    # 28,000 tiles, thousands of tensors skipped at once, then none: the search starts with a window of 4096
    "thousands": ([1 + (i * 7919) % 2048 for i in range(3000)] + [2048 * 13000 - 3, 77, 2048 * 40, 5] +
                  [2048 * (1 + i % 3) + i for i in range(700)] + [2048 * 9000, 2048, 1] + [900] * 1200, 50),
    # 20,250 tiles, 38 tensors skipped on average, up to 250: a window of 64, left where it does not reach
    "dozens": ([2048 * 40 - i for i in range(300)] + [1 + (i * 7919) % 2048 for i in range(250)] + [2048 * 40] * 200, 12)}


@pytest.mark.parametrize("many", sorted(MANY))
@pytest.mark.parametrize("tickets,stats", [(False, False), (True, False), (True, True)])
def test_a_unit_lies_any_number_of_tensors_after_the_last(ctx, tickets, stats, many):
    """Launches whose waves skip none, a few, dozens and thousands of tensors, drawn or not, against launches of a few."""
    sizes, few = MANY[many]
    plan = [(2 + i % 7, 2 + (i // 7) % 7) for i in range(len(sizes))]
    got, sums = [], []
    for group in (few, len(sizes)):
        sums.append([])
        m = model(ctx, sizes, plan, 64, 76)
        m.set_grads(1)
        ctx.set_schedule(1 if tickets and group > few else 2 ** 63)
        for a in range(0, len(sizes), group):
            which = list(range(a, min(a + group, len(sizes))))
            launch(ctx, m, 1, which, stats=stats)
            if stats:
                sums[-1] += [(s.count, s.g_sq_sum, s.g_absmax, s.v_absmax) for s in ctx.stats(len(which), m.stream)]
        ctx.set_schedule(0)
        torch.cuda.synchronize()
        nm = [m._code_words(n, b) for n, (b, _) in zip(sizes, plan)]
        nv = [m._code_words(n, b) for n, (_, b) in zip(sizes, plan)]
        got.append([torch.cat(m.param).view(torch.int32), torch.cat(m.m_scales).view(torch.int32), torch.cat(m.v_scales).view(torch.int32),
                    torch.cat([c[:k] for c, k in zip(m.m_codes, nm)]), torch.cat([c[:k] for c, k in zip(m.v_codes, nv)])])
        del m
    for x, y in zip(*got):
        assert torch.equal(x, y)
    for l, (x, y) in enumerate(zip(*sums)):  # fp64 in another order: n * 2^-53
        assert x[0] == y[0] and x[2:] == y[2:] and abs(x[1] - y[1]) <= 1e-12 * y[1], l


def test_many_small_tensors_are_not_walked_one_by_one(ctx):
    """4000 tensors of 16,384 elements, of which a wave skips hundreds between its tiles, against the same number of elements
    in four tensors, where there is nothing to skip (156 us against 125; a walk through all takes 849)."""
    best = {}
    for n in (4000, 4):
        m = model(ctx, [16384 * (4000 // n)] * n, [(8, 4)] * n, 128, 77)
        m.set_grads(1)
        for stats in (False, "grad"):
            for k in range(8):
                a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
                a.record()
                m.step(1, stats)
                b.record()
                torch.cuda.synchronize()
                if k > 1:
                    best[n, stats] = min(best.get((n, stats), 1e9), a.elapsed_time(b))
        if stats:
            ctx.stats(n, m.stream)
        del m
    for stats in (False, "grad"):
        assert best[4000, stats] < 2.5 * best[4, stats], best


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("sizes", [[1], [3, 2047, 2049], [1 + (i * 4093) % 9001 for i in range(700)], [2048 * 2500 + 5, 7, 2048 * 4, 2048 * 9000 - 1]])
def test_gradient_statistics_over_workgroup_ranges(ctx, sizes, dtype):
    """Tensors that begin and end anywhere in the range of tiles a workgroup of the gradient pass takes."""
    from workloads import configs
    from workloads.harness import DeviceModel
    w = configs.Workload(72, "gradients", [("t%d" % i, n) for i, n in enumerate(sizes)], 128, dtype, 1, "normal_per_tensor")
    m = DeviceModel(ctx, w, [(4, 4)] * len(sizes))
    m.set_grads(1)
    for _ in range(2):  # the second time on cleared accumulators
        ctx.grad_stats(m.tensors, 128, 1 if dtype == "bf16" else 0, m.stream)
        got = ctx.stats(len(sizes), m.stream)
    for l, n in enumerate(sizes):
        g = m.grad[l].double()
        # fp64 sums in some order: n * 2^-53 relative to the sum of absolute values
        bound = 1e-12
        assert got[l].count == n
        assert abs(got[l].g_sum - g.sum().item()) <= bound * g.abs().sum().item(), l
        assert abs(got[l].g_abs_sum - g.abs().sum().item()) <= bound * g.abs().sum().item(), l
        assert abs(got[l].g_sq_sum - (g * g).sum().item()) <= bound * (g * g).sum().item(), l
        assert got[l].g_absmax == g.abs().max().item(), l


def test_repack_chunks_over_job_boundaries(ctx):
    """A launch large enough for chunks of four tiles, whose jobs begin and end anywhere in a chunk, against one launch per job."""
    from paper_2604_06836_amd import binding
    sizes = [1 + (i * 7919) % 11000 for i in range(2500)] + [2048 * 3000 + 1]
    rng = np.random.default_rng(73)
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(73)
    jobs, dst, keep = [], [[], []], []
    for n in sizes:
        b0, b1, state = (int(x) for x in (rng.integers(2, 9), rng.integers(2, 9), rng.integers(0, 2)))
        tiles = (n + 2047) // 2048
        # (any codes will do: the conversion table has an entry for every code of the width)
        keep.append(torch.randint(-2 ** 31, 2 ** 31 - 1, (tiles * 64 * b0,), generator=gen, device="cuda:0", dtype=torch.int64).to(torch.int32))
        for d in dst:
            d.append(torch.full((tiles * 64 * b1,), -1, device="cuda:0", dtype=torch.int32))
        jobs.append((n, state, keep[-1].data_ptr(), b0, b1))
    assert sum((n + 2047) // 2048 for n in sizes) > 8192
    s = torch.cuda.current_stream().cuda_stream
    ctx.repack_many([(n, st, src, b0, d.data_ptr(), b1) for (n, st, src, b0, b1), d in zip(jobs, dst[0])], 64, s)
    for (n, st, src, b0, b1), d in zip(jobs, dst[1]):
        ctx.repack(n, 64, st, src, b0, d.data_ptr(), b1, s)
    torch.cuda.synchronize()
    for l, (x, y) in enumerate(zip(*dst)):
        assert torch.equal(x, y), l


@pytest.mark.parametrize("state,b0,b1", [(0, 3, 8), (1, 7, 4)])
def test_repack_beyond_the_caches(ctx, state, b0, b1):
    """369 MB of codes and more (read with the non-temporal hint) against two launches of half as much (read without)."""
    n, half = 2 ** 28 - 1001, 2 ** 27
    tiles = (n + 2047) // 2048
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(79)
    src = torch.randint(-2 ** 31, 2 ** 31 - 1, (tiles * 64 * b0,), generator=gen, device="cuda:0", dtype=torch.int64).to(torch.int32)
    dst = [torch.full((tiles * 64 * b1,), -1, device="cuda:0", dtype=torch.int32) for _ in range(2)]
    s = torch.cuda.current_stream().cuda_stream
    assert tiles * 256 * (b0 + b1) > 350 << 20
    ctx.repack(n, 64, state, src.data_ptr(), b0, dst[0].data_ptr(), b1, s)
    k = half // 2048 * 256
    ctx.repack(half, 64, state, src.data_ptr(), b0, dst[1].data_ptr(), b1, s)
    ctx.repack(n - half, 64, state, src.data_ptr() + k * b0, b0, dst[1].data_ptr() + k * b1, b1, s)
    torch.cuda.synchronize()
    assert torch.equal(*dst)


@pytest.mark.parametrize("eps", [1e-25, 2.0 ** -70, 1e-20, 1e-15, 1e-12, 0.5, 2.0 ** 39, 1e15])
def test_epsilon_inside_and_outside_the_short_forms_range(ctx, eps):
    """The short root and quotient take eps in [2^-70, 2^39], other values the IEEE routines: the oracle's bits either way,
    also where a block of v is all zero and den is eps alone."""
    from oracle import stq_oracle as oracle
    from workloads import configs
    from workloads.harness import DeviceModel
    hp = dict(configs.ADAM, eps=float(np.float32(eps)))
    sizes, plan = [2048 * 3 + 777, 5000], [(8, 4), (5, 8)]
    w = configs.Workload(74, "eps", [("a", sizes[0]), ("b", sizes[1])], 64, "fp32", 2, "normal_per_tensor", hparams=hp)
    m = DeviceModel(ctx, w, plan)
    th = [p.cpu().numpy().copy() for p in m.param]
    st = [oracle.State.zeros(n, 64, bm, bv) for n, (bm, bv) in zip(sizes, plan)]
    for t in (1, 2, 3):
        m.set_grads(t)
        m.grad[0][64:192] = 1e-30 if t == 1 else 0.0  # squares vanish: v = 0 where m is not
        m.grad[1][0:64] = 0.0
        m.step(t)
        torch.cuda.synchronize()
        for l in range(2):
            oracle.step(th[l], m.host_grad(l), st[l], **hp, t=t)
            p, mw, ms, vw, vs = m.host_state(l)
            assert np.array_equal(mw, oracle.pack(st[l].um, st[l].bm)) and np.array_equal(vw, oracle.pack(st[l].cv, st[l].bv))
            assert np.array_equal(ms, oracle.pad_scales(st[l].sm, st[l].numel, 64))
            assert np.array_equal(vs, oracle.pad_scales(st[l].sv, st[l].numel, 64))
            assert np.array_equal(p.view(np.uint32), th[l].view(np.uint32)), (t, l)
