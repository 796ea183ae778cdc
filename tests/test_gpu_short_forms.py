"""The short root, reciprocal and quotient of the step kernel, at the edges of what they are used for."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import paper_2604_06836_amd as stq
    c = stq.Context(0, 64)
    yield c
    c.close()


@pytest.mark.parametrize("bits", [(32, 32), (16, 16), (32, 4), (16, 8)])
def test_negative_zero_of_a_wide_first_moment(oracle, ctx, bits):
    """The short quotient of -0 is +0, the IEEE one -0: it shows in the sign of a parameter that is itself -0."""
    from workloads import configs
    from workloads.harness import DeviceModel
    n = 3 * 2048 + 100
    w = configs.Workload(75, "zeros", [("a", n)], 64, "fp32", 1, "normal")
    m = DeviceModel(ctx, w, [bits])
    st = oracle.State.zeros(n, 64, *bits)
    th = w.gen_param(0, "cpu").numpy().copy()
    th[::3] = -0.0
    th[1::7] = 0.0
    g = np.where(np.arange(n) % 2, np.float32(-0.0), np.float32(0.0)).astype(np.float32)
    g[5::11] = 1e-3  # (some blocks of v are not all zero)
    st.mw[:] = np.where(np.arange(n) % 5 < 3, np.float32(-0.0), np.float32(0.0))
    m.m_codes[0].copy_(torch.from_numpy(oracle.pack_wide(st.mw, bits[0]).view(np.int32)))
    m.param[0].copy_(torch.from_numpy(th))
    m.grad[0].copy_(torch.from_numpy(g))
    for t in (1, 2):
        m.step(t)
        torch.cuda.synchronize()
        oracle.step(th, g, st, **w.hparams, t=t)
        got = m.param[0].cpu().numpy()
        assert np.array_equal(got.view(np.uint32), th.view(np.uint32)), np.count_nonzero(got.view(np.uint32) != th.view(np.uint32))
        assert np.array_equal(m.m_codes[0].cpu().numpy().view(np.uint32), oracle.pack_wide(st.mw, bits[0]))


@pytest.mark.parametrize("K", [64, 128, 256])
@pytest.mark.parametrize("out", ["eps", "small", "mixed"])
def test_scales_and_eps_out_of_the_short_forms_range(oracle, ctx, K, out):
    """den from a table (widths up to 4, 5 and 6 at K = 64, 128 and 256) and from each element, by the IEEE routines: eps out
    of range, every scale of v out of range, and one block of a quarter in sixteen."""
    from workloads import configs
    from workloads.harness import DeviceModel
    plan = [(8, 2), (5, 3), (4, 4), (6, 5), (3, 6), (7, 7), (2, 8)]
    sizes = [4 * 2048 + 300 * i + 1 for i in range(len(plan))]
    hp = dict(configs.ADAM, eps=float(np.float32(1e-30 if out == "eps" else 1e-8)))
    w = configs.Workload(78, "range", [("t%d" % i, n) for i, n in enumerate(sizes)], K, "fp32", 2, "normal", hparams=hp)
    m = DeviceModel(ctx, w, plan)
    th = [p.cpu().numpy().copy() for p in m.param]
    st = [oracle.State.zeros(n, K, *b) for n, b in zip(sizes, plan)]
    for t in (1, 2, 3):
        m.set_grads(t)
        for l, g in enumerate(m.grad):
            if out == "small":  # v ~ 1e-32 < 2^-80
                g.mul_(1e-13)
            elif out == "mixed":
                g.view(-1)[64 * l:].view(-1)[:K] *= 1e-13
                g[2048:2048 + 512] *= 1e-13
        m.step(t)
        torch.cuda.synchronize()
        for l in range(len(plan)):
            oracle.step(th[l], m.host_grad(l), st[l], **hp, t=t)
            p, mw, ms, vw, vs = m.host_state(l)
            assert np.array_equal(mw, oracle.pack(st[l].um, st[l].bm)) and np.array_equal(vw, oracle.pack(st[l].cv, st[l].bv))
            assert np.array_equal(vs.view(np.uint32), oracle.pad_scales(st[l].sv, st[l].numel, K).view(np.uint32))
            assert np.array_equal(p.view(np.uint32), th[l].view(np.uint32)), (t, l)
    small = [float(np.min(s.sv[s.sv > 0])) for s in st]
    assert (out == "eps") == all(x > 2.0 ** -80 for x in small), small  # the cases really are what they claim
