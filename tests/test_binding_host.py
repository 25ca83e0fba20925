"""Host side of the binding: how wavelengths, phases and coefficients reach the library."""
import numpy as np
import pytest

from paper_2003_08960_amd import native


@pytest.mark.parametrize("values", [
    np.linspace(8e-7, 8.7e-7, 256), np.linspace(1, 2, 9)[::2], np.linspace(1, 2, 9)[::-1],
    np.arange(5), np.arange(3, dtype=np.uint8), np.float32([1.5, 2.25, 0.1]), np.array([]),
    np.array([1.0, 2.0], dtype=">f8"), [1, 2.5, np.float64(3)], (0.5,), np.array([True, False])])
def test_host_doubles_equal_the_elements(values):
    assert list(native.host_doubles(values)) == [float(v) for v in values]
    assert list(native.host_doubles(values, len(values))) == [float(v) for v in values]
    with pytest.raises(ValueError):
        native.host_doubles(values, len(values) + 1)


def test_host_doubles_copies_and_refuses_what_it_refused():
    a = np.array([1.0, 2.0])
    d = native.host_doubles(a)
    a[0] = 5.0
    assert list(d) == [1.0, 2.0]
    assert native.host_doubles(None) is None
    for bad in (np.ones((2, 2)), np.array(["a"]), ["x"]):
        with pytest.raises((TypeError, ValueError)):
            native.host_doubles(bad)
    with pytest.raises(TypeError):
        native.host_doubles(np.array(1.0))
