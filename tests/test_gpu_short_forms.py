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
