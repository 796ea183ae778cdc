"""Launches that write through (from 45,000 tiles on) give the bits of launches that do not, on both sides of the line: each of
the twelve kernels, at every width and block size and with ragged ends."""
import pytest

from test_gpu_units import compare, ctx, sizes_of  # noqa: F401 (a fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tiles", [44_999, 45_000])
@pytest.mark.parametrize("kind,dtype,K,stats", [("in_place", "bf16", 64, False), ("in_place", "fp32", 256, "grad"), ("transition", "bf16", 256, "grad"),
                                                ("transition", "fp32", 128, False), ("wide", "bf16", 128, False), ("wide", "fp32", 64, "grad"),
                                                ("in_place", "fp32", 128, False), ("in_place", "bf16", 128, "grad"), ("transition", "bf16", 64, False),
                                                ("transition", "fp32", 256, "grad"), ("wide", "fp32", 256, False), ("wide", "bf16", 64, "grad")])
def test_written_through(ctx, tiles, kind, dtype, K, stats):  # noqa: F811
    import torch
    compare(ctx, sizes_of(tiles, torch.cuda.get_device_properties(0).multi_processor_count), kind, dtype, K, stats)
