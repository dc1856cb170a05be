"""The way of calls that are captured, and of those that are too long for the short launch, at the lengths that other calls take the short
launch for: the suites of those lengths once more without it."""
import inspect

import pytest

import paper_2605_01708_amd as sz
import test_gpu_fuzz
import test_gpu_parity
import test_paged
import test_variants
from oracle import variants as ov

pytestmark = pytest.mark.gpu
SUITES = [test_gpu_fuzz.test_single_and_batch_calls_on_random_cases, test_gpu_fuzz.test_variant_calls_on_random_cases,
          test_gpu_fuzz.test_device_calibrated_batches_on_random_cases, test_gpu_parity.test_ragged_and_tiny_sizes,
          test_gpu_parity.test_all_bf16_bit_patterns, test_gpu_parity.test_all_e5m2_bit_patterns, test_gpu_parity.test_all_escape_and_no_escape,
          test_gpu_parity.test_escape_stress_outliers, test_gpu_parity.test_deterministic_and_workspace_reuse,
          test_gpu_parity.test_overflow_reports_needed_size, test_gpu_parity.test_batch_calls_match_the_oracle_item_by_item,
          test_gpu_parity.test_codebook_that_never_leaves_the_device, test_gpu_parity.test_batch_calibrated_on_the_device,
          test_gpu_parity.test_streaming_chunk_shape, test_paged.test_paged_pool_round_trip_matches_the_oracle_on_the_gathered_tensor,
          test_paged.test_table_entries_outside_the_pool_are_clamped, test_paged.test_batch_of_tensors_behind_one_block_table,
          test_variants.test_variant_overflow_and_bad_streams]


@pytest.fixture(autouse=True)
def no_short_launch():
    sz.internal_test_short(sz.INTERNAL_NO_SHORT)
    yield
    sz.internal_test_short()


@pytest.mark.parametrize("suite,dtype", [(f, d) for f in SUITES for d in (sz.BF16, sz.FP8_E5M2) if d == sz.BF16 or "dtype" in inspect.signature(f).parameters])
def test_without_the_short_launch(suite, dtype):
    given = {"dtype": dtype, "round_": 1}
    suite(**{name: given[name] for name in inspect.signature(suite).parameters})
