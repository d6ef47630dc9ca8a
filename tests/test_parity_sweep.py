"""The sweep of one step per launch, on the cases that pin its launch shapes and forms.

With a full workspace, matrices of rows of up to six entries step on tiles, where the
shape fields of a configuration have no effect.  Here the binding gives every call the
smallest workspace, which the sweep alone fits: block orders, rows and vectors per
thread, uniform values, 16-bit columns, the doubling form and seeded phases are the
sweep's again, with the bounds of the tests they come from.
"""
import pytest

from paper_2509_06525_amd import tbkpm
from tests.test_parity_batched import (test_batched_fp64_moments_per_structure,  # noqa: F401
                                       test_xcd_mapping_is_bitwise_neutral)
from tests.test_parity_doubling import (test_c32_doubling_dos_within_1e_4, test_fp64_doubling_every_shape,  # noqa: F401
                                        test_fp64_doubling_matches_direct_oracle,
                                        test_fp64_doubling_onsite_and_shift)
from tests.test_parity_launch import (test_c32_shapes_agree, test_fp64_every_shape_matches_oracle,  # noqa: F401
                                      test_xcd_block_orders_are_bitwise_neutral)
from tests.test_parity_resume import (test_split_run_is_bitwise_the_one_shot_run,  # noqa: F401
                                      test_split_run_with_another_launch_shape)
from tests.test_parity_seeded import test_seeded_c32_dos_and_row_order, test_seeded_fp64_moments_match_oracle  # noqa: F401
from tests.test_parity_uniform import (test_compact_columns_bitwise, test_four_rows_per_thread,  # noqa: F401
                                       test_pristine_uniform_values_bitwise, test_uniform_values_with_doubling,
                                       test_uniform_values_with_padding_rows)

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def smallest_workspace(monkeypatch):
    """Every workspace the binding or a test asks for is the sweep's, below that of the tiles
    (the persistent launch and doubling runs of few moments, which are not offered tiles, have
    one size)."""
    asked = []

    def least_of(full, least):
        def size(H, R, M, precision, config=None, *args, **kw):
            n = least(H, R, M, precision, config, *args, **kw)
            swept = config is not None and (config.persistent or (config.doubling and M < 8))
            assert swept or n < full(H, R, M, precision, config, *args, **kw)
            asked.append(n)
            return n
        return size

    monkeypatch.setattr(tbkpm, "workspace_size", least_of(tbkpm.workspace_size, tbkpm.least_workspace_size))
    monkeypatch.setattr(tbkpm, "workspace_size_batched",
                        least_of(tbkpm.workspace_size_batched, tbkpm.least_workspace_size_batched))
    yield
    assert asked and tbkpm.last_form()[0] == 0
