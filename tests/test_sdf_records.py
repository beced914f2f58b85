"""The face records of an index SDF's update, on the host: room only where they are used."""

import pytest

from paper_2606_00444_amd import sdf
from paper_2606_00444_amd._lib import MguError


@pytest.mark.parametrize("n_faces,k,dims,used", [
    (40000, 4, (64, 64, 64), True), (40000, 4, (32, 64, 64), True), (40000, 4, (31, 64, 64), False),
    (40000, 3, (64, 64, 64), False), (40000, 5, (128, 128, 128), False), (500000, 1, (128, 64, 64), True),
    (500000, 1, (64, 64, 64), False), (1 << 20, 4, (64, 64, 64), True), ((1 << 20) + 1, 4, (64, 64, 64), False),
    (0, 4, (64, 64, 64), False)])
def test_records_are_held_where_they_are_used(n_faces, k, dims, used):
    assert sdf.records_bytes(n_faces, k, dims) == (48 * n_faces if used else 0)


def test_bad_arguments():
    for args in ((-1, 4, (8, 8, 8)), (10, 0, (8, 8, 8)), (10, 65, (8, 8, 8)), (10, 4, (8, 0, 8))):
        with pytest.raises(MguError):
            sdf.records_bytes(*args)
