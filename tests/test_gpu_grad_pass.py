"""The gradients' statistics of stq_grad_stats at the edges of its loads (16 or 8 bytes a lane, whole tiles apart from ragged
ones) and of its division of the work, against numpy's float64; and their
read-back, which waits for the stream."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

SIZES = {
    # one tile a wave: every remainder of a load, of a row, of a tile
    "edges": [1, 2, 3, 4, 5, 7, 8, 9, 255, 256, 257, 259, 1023, 1024, 1791, 2044, 2045, 2047, 2048, 2049, 2051, 4095, 4096, 4099],
    # several tiles a wave: waves that end in different tensors of their workgroup's range, ragged tiles between whole ones
    "ranges": [700_001, 2048 * 3, 5, 2048 * 1999 + 1, 2048 * 41 + 2046, 1, 2_500_003] + [2048 * 2 + 7 * k for k in range(9)],
    "one": [2048 * 4100],
}


@pytest.mark.parametrize("dtype", ["fp32", "bf16"])
@pytest.mark.parametrize("which", SIZES)
def test_edges_of_the_gradient_pass(which, dtype):
    import paper_2604_06836_amd as stq
    from workloads import configs
    from workloads.harness import DeviceModel
    sizes = SIZES[which]
    ctx = stq.Context(0, 64)
    w = configs.Workload(97, "gpass-%s-%s" % (which, dtype), [("t%d" % i, n) for i, n in enumerate(sizes)], 128, dtype, 1, "normal_per_tensor")
    m = DeviceModel(ctx, w, [(4, 4)] * len(sizes))
    m.set_grads(1)
    for _ in range(2):  # the second call finds the accumulators cleared, and gradients of twice the size
        ctx.grad_stats(m.tensors, w.K, 1 if dtype == "bf16" else 0, m.stream)
        got = ctx.stats(len(sizes), m.stream)
        for l, g in enumerate(got):
            x = m.grad[l].double().cpu().numpy()
            total = np.abs(x).sum()
            assert g.count == sizes[l] and g.g_absmax == np.abs(x).max(), l
            # fp64 additions in another order: no chain is longer than 3000 (a lane's elements, the lanes, the workgroups),
            # 3000 * 2^-53 = 3.4e-13 of the sum of absolute values
            for a, b, scale in ((g.g_sum, x.sum(), total), (g.g_abs_sum, total, total), (g.g_sq_sum, (x * x).sum(), (x * x).sum())):
                assert abs(a - b) <= 1e-12 * scale, (l, a, b)
        for g in m.grad:
            g.mul_(2)  # exact in both types
    ctx.close()


@pytest.mark.parametrize("busy", [False, True])
def test_read_back(busy):
    """Calls for more tensors and for fewer than the call before, each with other gradients; also behind some milliseconds of
    work.  A call returns when its stream is idle."""
    import paper_2604_06836_amd as stq
    from workloads import configs
    from workloads.harness import DeviceModel
    counts = [1, 16, 17, 40, 33, 32, 1, 40]
    ctx = stq.Context(0, 40)
    w = configs.Workload(98, "read-back", [("t%d" % i, 100 + i) for i in range(40)], 64, "fp32", 1, "normal_per_tensor")
    m = DeviceModel(ctx, w, [(4, 4)] * 40)
    m.set_grads(1)
    x = [g.double().abs().cpu().numpy() for g in m.grad]
    big = torch.zeros(1 << 30, dtype=torch.uint8, device="cuda") if busy else None
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        for call, n in enumerate(counts):
            for _ in range(40 if busy else 0):  # 40 passes over 1 GiB: 10 ms
                big.add_(1)
            for g in m.grad:
                g.mul_(2)  # exact
            ctx.grad_stats((type(m.tensors[0]) * n)(*m.tensors[:n]), w.K, 0, m.stream)
            got = ctx.stats(n, m.stream)
            assert side.query(), call
            for l, g in enumerate(got):
                y = x[l] * 2.0 ** (call + 1)
                assert g.count == y.size and g.g_absmax == y.max() and abs(g.g_abs_sum - y.sum()) <= 1e-12 * y.sum(), (call, l)
    ctx.close()
