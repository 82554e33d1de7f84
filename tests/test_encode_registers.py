"""The one-launch encoder's kernels spill no vector register, in any stored form: one that spills needs scratch memory, and the
launch of a kernel that does takes 1 to 2 us more, 2 % of one layer's chunk."""
from test_kernel_registers import spilled  # noqa: F401  (fixture)


def test_the_one_launch_encoder_does_not_spill(spilled):  # noqa: F811
    kernels = {k: v for k, v in spilled.items() if k.startswith("lloyd_kernel<")}
    assert len(kernels) >= 12
    assert not any(kernels.values()), kernels
