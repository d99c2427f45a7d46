"""Which distances of the flat and peer buffers are staggered: within 20 MiB (five to eight replicas: 6) of a multiple of 256 MiB."""
import pytest

from paper_2502_11058_amd.harness import stagger


@pytest.mark.parametrize("mib,many,few", [(2, False, False), (20, False, False), (234, False, False), (236, True, False), (248, True, False), (250, True, True),
                                          (256, True, True), (262, True, True), (264, True, False), (276, True, False), (278, False, False),
                                          (384, False, False), (490, False, False), (492, True, False), (514, True, True), (534, False, False),
                                          (3840 + 20, True, False), (3840 + 22, False, False)])
def test_distances(mib, many, few):
    for replicas, yes in ((9, many), (8, few), (5, few), (4, False)):
        assert stagger(mib << 20, replicas) == stagger((mib << 20) - 1, replicas) == (640 << 10 if yes else 0)
