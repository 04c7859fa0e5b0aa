"""bench.py's names of profiled kernels, on the CPU."""
import os
import sys

sys.path.insert(0, os.path.dirname(os.path.dirname(os.path.abspath(__file__))))


def test_the_combine_is_one_kernel():
    # its parameters are the head size and the type of the operands it writes:
    # both passes launch <128, 0> in the bf16 step, and <128, 1> is fp32's
    import bench
    assert bench.profile_name("void la::combine_kernel<128, 0>(float const*, int, ...)") == "combine"
    assert bench.profile_name("void la::combine_kernel<128, 1>(float const*, int, ...)") is None
