"""The streaming kernel and the kernels that take the activations through LDS at the sizes where they can go wrong, by the tuning build with the batch and tile
kernels left out: the library gives groups as small as these to those two, so the tests of grouped calls reach the other kernels' ragged batches, split
rows, re-planned workgroups and short steps only here."""
import pytest

import test_gpu_grouped_rounds as rounds
import test_gpu_grouped_small as small
import test_gpu_parity as parity
import test_gpu_rows_w3 as rows_w3
from test_gpu_parity import awq, small_group                       # noqa: F401 (fixtures)
from tuning_build import tuning_build

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def without_the_batch_and_tile_kernels():
    with tuning_build(AWQ_FEW=0):
        yield


def parameters(test):
    """The parametrization of another file's test."""
    def decorate(f):
        for mark in test.pytestmark:
            if mark.name == "parametrize":
                f = pytest.mark.parametrize(*mark.args, **mark.kwargs)(f)
        return f
    return decorate


@parameters(rounds.test_one_round_of_workgroups)
def test_rounds(bits, M, shapes):
    rounds.test_one_round_of_workgroups(bits, M, shapes)


@parameters(small.test_grouped_launch_at_five_to_seven_tokens)
def test_five_to_seven_tokens(M, shapes):
    small.test_grouped_launch_at_five_to_seven_tokens(M, shapes)


@parameters(rows_w3.test_w3_rows_launch_against_the_oracle)
def test_w3_rows(M, shapes):
    rows_w3.test_w3_rows_launch_against_the_oracle(M, shapes)


@pytest.mark.parametrize("M", range(1, 17))
def test_every_m(awq, small_group, M):                             # noqa: F811
    parity.test_multi_every_m(awq, small_group, M)


@pytest.mark.parametrize("test", [parity.test_multi_exact_and_deterministic_on_integer_data, parity.test_multi_more_than_four_tokens_ragged_shapes,
                                  parity.test_w3_grouped_small_every_m_and_integer_exactness])
def test_groups(awq, test):                                        # noqa: F811
    test(awq)
