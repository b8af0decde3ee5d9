"""The library builds that the GPU tests of the exchange between workgroups run (tests/exchange_builds.py): made here, where there
is a compiler and no GPU needed, so that those tests find them."""
import ctypes
import os

import pytest

from paper_2503_05096_amd import build
from tests import exchange_builds


def test_sources_that_exchange_words_are_found():
    names = {os.path.basename(s) for s in build._sources() if build._includes(s, "part_exchange.h")}
    assert {"accept_parts.hip", "accept_shared.hip", "draft_parts.hip", "tree_fast.hip"} <= names
    assert "attn_mfma.hip" not in names


@pytest.mark.parametrize("name", sorted(exchange_builds.DEFINES))
def test_build_of_the_current_sources(name):
    import torch  # noqa: F401  (the HIP runtime of this process)
    L = ctypes.CDLL(exchange_builds.ensure(name))
    assert L.adaspec_version() > 0
    assert os.path.basename(exchange_builds.path(name)).split("_")[-1] == build.source_key(exchange_builds.DEFINES[name]) + ".so"
