"""Channel groups that the autotuner times: the library's own choice once, not
again under its explicit number."""
import pytest

from paper_2511_22793_amd import serve


@pytest.mark.parametrize("fc,groups", [(1, [0]), (2, [0]), (3, [0, 1]), (8, [0]), (10, [0, 2]), (24, [0, 8]),
                                       (32, [0, 8, 16, 32]), (128, [0, 8, 16, 32])])
def test_candidates(fc, groups):
    assert serve.group_candidates(fc) == groups
