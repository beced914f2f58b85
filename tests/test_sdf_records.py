"""The face records of an index SDF's update, on the host: room only where they are used."""

import pytest

from paper_2606_00444_amd import sdf
from paper_2606_00444_amd._lib import MguError


@pytest.mark.parametrize("n_faces,k,dims,used", [
    (40000, 4, (64, 64, 64), True), (40000, 4, (63, 64, 64), False), (500, 4, (64, 64, 64), True),
    (40000, 3, (64, 64, 64), False), (40000, 5, (128, 128, 128), False),
    (4096, 1, (128, 128, 128), True), (4095, 1, (128, 128, 128), False), (500000, 1, (127, 128, 128), False),
    (500, 2, (96, 128, 64), True), (40000, 2, (95, 128, 64), False),
    (500000, 8, (64, 32, 32), True), (500, 8, (63, 32, 32), False),
    (1 << 20, 4, (64, 64, 64), True), ((1 << 20) + 1, 4, (64, 64, 64), False), (0, 4, (64, 64, 64), False)])
def test_records_are_held_where_they_are_used(n_faces, k, dims, used):
    assert sdf.records_bytes(n_faces, k, dims) == (48 * n_faces if used else 0)


def test_bad_arguments():
    for args in ((-1, 4, (8, 8, 8)), (10, 0, (8, 8, 8)), (10, 65, (8, 8, 8)), (10, 4, (8, 0, 8))):
        with pytest.raises(MguError):
            sdf.records_bytes(*args)
