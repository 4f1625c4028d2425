"""The Python binding on the host: what it hands to the library."""
import ctypes

import pytest

from paper_2609_33570_amd import hilore

FIELDS = [name for name, _ in hilore.hilore_unit_desc._fields_]


class Longer(hilore.hilore_unit_desc):
    _fields_ = [("tag", ctypes.c_int64)]


class Renamed(hilore.hilore_unit_desc):
    pass


def values(i):
    return tuple((1 << 20) + 4096 * i + 256 * k for k in range(6)) + (10 + i, 128 * (i + 1), 128 * (i + 2))


@pytest.mark.parametrize("n", [0, 1, 3, 4, 5, 17])
@pytest.mark.parametrize("make", [
    lambda i: hilore.hilore_unit_desc(*values(i)),
    lambda i: Longer(*values(i), 7),
    lambda i: Renamed(*values(i)),
    values,
    lambda i: (hilore.hilore_unit_desc(*values(i)), Longer(*values(i), 7), values(i))[i % 3],
], ids=["plain", "longer", "renamed", "tuple", "mixed"])
def test_descriptor_array(make, n):
    """Every form of descriptor that a ctypes array takes arrives unchanged, in any number."""
    arr, count = hilore._desc_array([make(i) for i in range(n)])
    assert count == n and ctypes.sizeof(arr) == 72 * max(1, n)
    for i in range(n):
        assert tuple(getattr(arr[i], f) for f in FIELDS) == values(i)


@pytest.mark.parametrize("n", [1, 5])
def test_descriptor_array_refuses_other_types(n):
    with pytest.raises(TypeError):
        hilore._desc_array([ctypes.c_int64(3)] * n)
