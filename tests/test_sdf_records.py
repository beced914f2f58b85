"""The face records of an index SDF's update, on the host: room only where they are used."""

import pytest

from paper_2606_00444_amd import sdf
from paper_2606_00444_amd._lib import MguError


def _cases():
    # stored ids (in 2^16) from which records are used, by k and by meshes of 2,047, 2,048, 65,536,
    # 65,537, 262,144 and 262,145 faces
    faces = (2047, 2048, 65536, 65537, 262144, 262145)
    for k, least in ((1, (None, 13, 13, 24, 24, 16)), (2, (24, 8, 8, 18, 18, 16)), (4, (8, 8, 8, 14, 14, 8)), (8, (8,) * 6)):
        for nf, ids in zip(faces, least):
            if ids is None:
                yield nf, k, (256, 256, 256), False
                continue
            layer = (ids << 16) // k // 64                # nodes in 64 layers
            yield nf, k, (layer // 128, 128, 64), True
            yield nf, k, (layer // 128 - 1, 128, 64), False
    for nf, k in ((40000, 3), (40000, 5), (0, 4)):
        yield nf, k, (128, 128, 128), False
    yield 1 << 20, 4, (64, 64, 64), True                  # as many ids as faces
    yield (1 << 20) + 1, 4, (64, 64, 64), False


@pytest.mark.parametrize("n_faces,k,dims,used", list(_cases()))
def test_records_are_held_where_they_are_used(n_faces, k, dims, used):
    assert sdf.records_bytes(n_faces, k, dims) == (48 * n_faces if used else 0)


def test_bad_arguments():
    for args in ((-1, 4, (8, 8, 8)), (10, 0, (8, 8, 8)), (10, 65, (8, 8, 8)), (10, 4, (8, 0, 8))):
        with pytest.raises(MguError):
            sdf.records_bytes(*args)
