"""Half and quarter tiles give the same bits, on both sides of every line at which the launch changes its units, its order, its
counters or its workgroups: each tensor by itself is a launch of quarter tiles (which the other GPU tests compare with the
oracle), all together one of the size asked for."""
import numpy as np
import pytest
import torch

from test_gpu_schedules import launch, model, outputs

pytestmark = pytest.mark.gpu

WIDTHS = {"in_place": [2, 3, 4, 5, 6, 7, 8], "transition": [2, 3, 4, 5, 6, 7, 8], "wide": [3, 4, 5, 8, 16, 32]}


@pytest.fixture(scope="module")
def ctx():
    import paper_2604_06836_amd as stq
    c = stq.Context(0, 2048)
    yield c
    c.close()


def sizes_of(tiles, n_cu):
    """Tensors of at most n_cu tiles (quarters with statistics too), ragged in every quarter of their last tile."""
    out = []
    while tiles:
        nt = min(tiles, 1 + (n_cu - 57 * (len(out) % 4)) % n_cu)
        out.append(nt * 2048 - [0, 1, 300, 511, 512, 700, 1024, 1500, 1536, 2047][len(out) % 10])
        tiles -= nt
    return out


# per CU: statistics in halves above 1 tile, plain halves above 6, all at once up to 8, drawn from 16 (fp32) or 24 on
@pytest.mark.parametrize("per_cu,more", [(1, 1), (6, 0), (6, 1), (8, 0), (8, 1), (16, 0), (24, 0), (24, 77)])
@pytest.mark.parametrize("kind,dtype,K,stats", [("in_place", "bf16", 64, False), ("in_place", "fp32", 256, True), ("transition", "fp32", 128, False),
                                                ("transition", "bf16", 64, "grad"), ("wide", "fp32", 64, False), ("wide", "bf16", 128, True)])
def test_halves_and_quarters_give_the_same_bits(ctx, per_cu, more, kind, dtype, K, stats):
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    compare(ctx, sizes_of(per_cu * n_cu + more, n_cu), kind, dtype, K, stats)


# wide states with fp32 gradients: two workgroups per CU below 30,000 tiles, one from there on; eight counters below 100,000
# tiles, then one
@pytest.mark.parametrize("tiles,kind,dtype,K,stats", [(29_999, "wide", "fp32", 64, False), (30_000, "wide", "fp32", 64, False),
                                                      (30_000, "wide", "fp32", 256, True), (99_999, "in_place", "bf16", 128, False),
                                                      (100_000, "in_place", "bf16", 128, False), (100_000, "in_place", "fp32", 64, "grad")])
def test_lines_of_large_launches(ctx, tiles, kind, dtype, K, stats):
    compare(ctx, sizes_of(tiles, torch.cuda.get_device_properties(0).multi_processor_count), kind, dtype, K, stats)


# with statistics, above one tile per CU: quarters below 16 tiles a tensor on average
@pytest.mark.parametrize("stats", [True, "grad"])
@pytest.mark.parametrize("tiles", [15, 16])
def test_statistics_of_small_tensors(ctx, tiles, stats):
    compare(ctx, [2048 * tiles - (l * 97) % 2048 for l in range(60)], "in_place", "fp32", 128, stats)


def compare(ctx, sizes, kind, dtype, K, stats):
    w = WIDTHS[kind]
    plan = [(w[i % len(w)], w[(i // len(w) + 2 * i) % len(w)]) for i in range(len(sizes))]
    new = [(b, a) for a, b in plan] if kind != "in_place" else None
    got, sums = [], []
    for together in (False, True):
        m = model(ctx, sizes, plan, K, 90, dtype)
        for lst in (m.m_codes, m.v_codes):  # nothing undefined behind a state narrower than its buffer
            for l, buf in enumerate(lst):
                buf[m._code_words(sizes[l], plan[l][0 if lst is m.m_codes else 1]):] = 0
        for s in m._spare.values():
            s.zero_()
        m.set_grads(1)
        sums.append([])
        for t in (1, 2):
            for g in [list(range(len(sizes)))] if together else [[l] for l in range(len(sizes))]:
                launch(ctx, m, t, g, new, stats)
                if stats:
                    sums[-1] += [(s.count, s.g_absmax, s.m_absmax, s.v_absmax, s.g_sum, s.m_sum, s.g_abs_sum, s.g_sq_sum, s.m_sq_sum, s.m_err_sq,
                                  s.v_sum, s.v_sq_sum, s.v_err_sq) for s in ctx.stats(len(g), m.stream)]
        got.append(outputs(m))
        del m
    for a, b in zip(*got):
        for l, (x, y) in enumerate(zip(a, b)):
            assert torch.equal(x.view(torch.int32), y.view(torch.int32)), l
    for i, (a, b) in enumerate(zip(*sums)):
        assert a[:4] == b[:4], i
        # Sums of the same numbers in another order, in fp64 (those of the moments' squares, of v and of the errors over eight
        # elements of a lane in fp32 first, the same eight in halves and quarters).  No chain of additions is longer than 2000
        # (a lane's elements, its units, the waves, the workgroups): 2000 * 2^-53 = 2.2e-13 of the sum of absolute values,
        # for that of the first moments at most sqrt(n * sum of squares).
        assert abs(a[4] - b[4]) <= 1e-12 * a[6] and abs(a[5] - b[5]) <= 1e-12 * np.sqrt(a[0] * a[8]), i
        for x, y in zip(a[6:], b[6:]):
            assert abs(x - y) <= 1e-12 * x, i
