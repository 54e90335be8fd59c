"""Which sources the profiles' figures belong to (CPU)."""
import pytest

from paper_1912_12675_amd.rocprof_summary import kernel_sources

CSRC = "paper_1912_12675_amd/csrc/"


@pytest.mark.parametrize("kernel, sources", [
    ("conv3x3_direct<32, 1, 8, 16, 1, 4, 4, false, 1, 0, false>", ["direct.hip", "internal.h"]),
    ("conv3x3_wgrad<1, 32, 16, 1, 1, 4, 1, 2, false, 2, true>", ["wgrad.hip", "internal.h"]),
    ("reduce_splits<4, 1>", ["conv.hip", "internal.h"]),
    ("gemm_rows<false, 1, 4>", ["fc.hip", "internal.h", "split.h"]),
    ("gemm_split<3, 64, 64, 2, 2, 1, 2, true, false>", ["fc.hip", "internal.h", "split.h"]),
    ("conv_split<1, 32, 256, 4, 1, 2, 2>", ["gconv.hip", "internal.h", "split.h"]),
    ("conv_split_wgrad<1, 64, 2, 1, 1, 5, 16>", ["gwgrad.hip", "internal.h", "split.h"]),
    ("chan_sums_wide<2, 4>", ["bn.hip", "internal.h"]),
    ("bn_stats_partials_k", ["ops.hip", "internal.h"]),
    ("softmax_xent_k", ["ops.hip", "internal.h"]),
])
def test_kernel_sources_name_the_file_that_defines_it(kernel, sources):
    assert kernel_sources(kernel) == [CSRC + f for f in sources]


def test_an_unknown_kernel_is_refused():
    with pytest.raises(SystemExit):
        kernel_sources("no_such_kernel")
