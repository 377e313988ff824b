"""Ranges and defaults of library options (CPU)."""
import pytest

import paper_1312_0526_amd as mx


@pytest.mark.parametrize("key,default,good,bad", [("shared_rounds", 24, (0, 24), (-1, 25)),
                                                  ("group_wait", 20, (0, 1000), (-1, 1001)),
                                                  ("group_joins", 0, (0,), (-1, 1))])
def test_option_ranges(key, default, good, bad):
    assert mx.get_option(key) == default
    try:
        for v in good:
            mx.set_option(key, v)
            assert mx.get_option(key) == v
        for v in bad:
            with pytest.raises(mx.MphxError):
                mx.set_option(key, v)
            assert mx.get_option(key) == good[-1]
    finally:
        mx.set_option(key, default)
