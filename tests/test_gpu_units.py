"""Half and quarter tiles give the same bits, on both sides of every line at which the launch changes its units or its order:
each tensor by itself is a launch of quarter tiles (which the other GPU tests compare with the oracle), all together one of the
size asked for."""
import numpy as np
import pytest
import torch

from test_gpu_schedules import launch, model, outputs

pytestmark = pytest.mark.gpu

WIDTHS = {"in_place": [2, 3, 4, 5, 6, 7, 8], "transition": [2, 3, 4, 5, 6, 7, 8], "wide": [3, 4, 5, 8, 16, 32]}


@pytest.fixture(scope="module")
def ctx():
    import paper_2604_06836_amd as stq
    c = stq.Context(0, 256)
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
    sizes = sizes_of(per_cu * n_cu + more, n_cu)
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
                    sums[-1] += [(s.count, s.g_absmax, s.m_absmax, s.v_absmax, s.g_sq_sum, s.m_sq_sum, s.v_err_sq) for s in ctx.stats(len(g), m.stream)]
        got.append(outputs(m))
        del m
    for a, b in zip(*got):
        for l, (x, y) in enumerate(zip(a, b)):
            assert torch.equal(x.view(torch.int32), y.view(torch.int32)), l
    for i, (a, b) in enumerate(zip(*sums)):
        assert a[:4] == b[:4], i
        # non-negative terms: fp64 in another order, n * 2^-53; the moments' in fp32 over eight rows of a lane and eight lanes
        assert abs(a[4] - b[4]) <= 1e-12 * a[4], i
        assert np.allclose(a[5:], b[5:], rtol=1e-5, atol=2048 * n_cu * 1.2e-38), i
