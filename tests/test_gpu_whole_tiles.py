"""The kernels of half tiles against the oracle.  Launches as small as the other parity tests use take quarter tiles; here a
filler tensor makes them large enough for halves, with tickets drawn ("tickets") or every workgroup's own ("stripes", on 25,400
tiles).  The filler itself is compared with a launch of its own, whose tickets are its workgroups' own.  (The names here are older
than half tiles.)"""
import numpy as np
import pytest
import torch

from test_gpu_parity import assert_stats_close, assert_tensor_parity

pytestmark = pytest.mark.gpu

NARROW = [(bm, bv) for bm in range(2, 9) for bv in range(2, 9)]
WIDE = [(bm, bv) for bm in (2, 3, 4, 5, 6, 7, 8, 16, 32) for bv in (2, 3, 4, 5, 6, 7, 8, 16, 32) if max(bm, bv) >= 16]
FILL = [(5, 3), (6, 7)]


@pytest.fixture(scope="module")
def ctx():
    import paper_2604_06836_amd as stq
    c = stq.Context(0, 64)
    yield c
    c.close()


def assert_stats(g, o, stats, tag):
    if stats == "grad":  # the moments' fields stay 0
        for f in ("m_sum", "m_sq_sum", "m_err_sq", "v_sum", "v_sq_sum", "v_err_sq", "m_absmax", "v_absmax"):
            assert getattr(g, f) == 0.0, (tag, f)
        for f in ("g_sum", "g_abs_sum", "g_sq_sum"):
            assert abs(getattr(g, f) - getattr(o, f)) <= 1e-12 * (o.g_abs_sum if f == "g_sum" else getattr(o, f)), (tag, f)
        assert g.count == o.count and g.g_absmax == o.g_absmax, tag
    else:
        assert_stats_close(g, o, tag)


CASES = [("tickets", kind, dtype) for kind in ("in_place", "transition", "wide") for dtype in ("fp32", "bf16")] + \
    [("stripes", kind, "bf16") for kind in ("in_place", "transition")]


@pytest.mark.parametrize("K", [64, 128, 256])
@pytest.mark.parametrize("schedule,kind,dtype", CASES)
def test_whole_tiles_against_the_oracle(oracle, ctx, schedule, kind, dtype, K):
    """Every pair of widths (in place, or every pair as the stored and as the written one), ragged ends, every choice of
    statistics."""
    from workloads import configs
    from workloads.harness import DeviceModel
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    fill = [(24 * n_cu + 300) * 2048 + 5] if schedule == "tickets" else [12700 * 2048 + 5, 12700 * 2048 - 900]
    pairs = WIDE if kind == "wide" else NARROW
    rng = np.random.default_rng(K)
    small = [int(rng.integers(0, 3)) * 2048 + int(rng.integers(1, 2048)) for _ in pairs]
    F = len(fill)
    names = [("t%d" % i, n) for i, n in enumerate(fill + small)]
    # (with a spare buffer for every state: a width change then writes the other one)
    w = configs.Workload(81, "whole", names, K, dtype, 1, "normal_per_tensor")
    m = DeviceModel(ctx, w, FILL[:F] + pairs, spare_width=32 if kind == "wide" else 8)
    alone = [DeviceModel(ctx, configs.Workload(82, "fill%d" % i, [("f", n)], K, dtype, 1, "normal_per_tensor"), [FILL[i]], spare_width=8)
             for i, n in enumerate(fill)]
    for i, a in enumerate(alone):
        a.param[0].copy_(m.param[i])
    th = [p.cpu().numpy().copy() for p in m.param[F:]]
    st = [oracle.State.zeros(n, K, *p) for n, p in zip(small, pairs)]
    rounds = [(change, stats) for change in {"in_place": (False,), "transition": (True,), "wide": (False, True)}[kind]
              for stats in (False, True, "grad")]
    for t, (change, stats) in enumerate(rounds, 1):
        m.set_grads(t)
        # the small tensors' new widths: pair i goes to pair i + 11, the filler's change places
        plan = m.plan[F:]
        new = plan[11:] + plan[:11]
        fill_new = [(b, a) for a, b in m.plan[:F]]
        ctx.set_schedule(1 if schedule == "tickets" else 2 ** 63)
        if change:
            m.step_transition(t, fill_new + new, stats)
        else:
            m.step(t, stats)
        torch.cuda.synchronize()
        got = ctx.stats(len(names), m.stream) if stats else None
        ctx.set_schedule(2 ** 63)
        tag = "%s step %d" % (kind, t)
        for l in range(len(small)):
            args = (th[l], m.host_grad(F + l), st[l]) + (new[l] if change else ())
            s = (oracle.step_transition if change else oracle.step)(*args, **w.hparams, t=t, want_stats=bool(stats))
            assert_tensor_parity(oracle, _Tail(m, F), l, th[l], st[l], tag)
            if stats:
                assert_stats(got[F + l], s, stats, "%s tensor %d" % (tag, l))
        for i, a in enumerate(alone):
            a.grad[0].copy_(m.grad[i])
            if change:
                a.step_transition(t, [fill_new[i]], stats)
            else:
                a.step(t, stats)
            if stats:
                assert_stats(got[i], ctx.stats(1, a.stream)[0], stats, "%s filler" % tag)
            torch.cuda.synchronize()
            words = [m._code_words(fill[i], b) for b in m.plan[i]]
            for x, y, k in ((m.param[i], a.param[0], None), (m.m_scales[i], a.m_scales[0], None), (m.v_scales[i], a.v_scales[0], None),
                            (m.m_codes[i], a.m_codes[0], words[0]), (m.v_codes[i], a.v_codes[0], words[1])):
                assert torch.equal(x.view(torch.int32)[:k], y.view(torch.int32)[:k]), (tag, i)
    ctx.set_schedule(0)


class _Tail:
    """The tensors of a model from index F on."""

    def __init__(self, m, F):
        self.m, self.F = m, F

    def host_state(self, l):
        return self.m.host_state(self.F + l)
