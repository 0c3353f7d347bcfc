"""The orbit search on labels of 2 to 5 bits per site, by the walk over digit
planes (groups of more than 16 elements) and by the images of all elements
(up to 16), with numbers of sites that leave one, two or three of a four-site
chunk, with and without the spin flip: representatives, connecting elements,
indices and products as in test_gpu_orbit.py."""
import pytest

import test_gpu_orbit as orbit

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,keep,two_s,two_M,flip", [
    ("petersen", None, 3, 24, False), ("petersen", None, 5, 42, False), ("petersen", None, 8, 72, False),
    ("petersen", None, 17, 162, False), ("ring7", None, 8, 48, False), ("ring7", None, 17, 111, False),
    ("ring6", None, 3, 0, True), ("ring5", None, 2, 0, True), ("ring9", None, 2, 8, False), ("ring11", None, 1, 1, False),
])
def test_orbit_search_by_digits(name, keep, two_s, two_M, flip):
    orbit.test_orbit_search(name, keep, two_s, two_M, flip)
