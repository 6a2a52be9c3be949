"""The harnesses refuse a built library that is older than any file it is compiled from."""
import os

import pytest

from paper_2603_08343_amd import build


@pytest.mark.parametrize("built,source", [(build.LIB, f) for f in ("wht_affine.hip", "wht_device.h", "wht_plan.h", "wht_route.h", "wht_validate.h")] +
                         [(build.POISON_LIB, "wht_validate.h"), (build.MARSHAL_LIB, "torch_marshal.cpp"),
                          (build.LIB, build.HEADER), (build.MARSHAL_LIB, build.HEADER),
                          (build.ROUTE_LIB, "wht_route.h"), (build.ROUTE_LIB, "route_query.cpp")])
def test_an_older_library_is_refused(built, source, monkeypatch):
    source = os.path.join(build.HERE, "csrc", source)          # an absolute path stays what it is
    real = os.path.getmtime
    build.ensure_built()
    monkeypatch.setattr(os.path, "getmtime", lambda f: real(source) - 1.0 if f == built else real(f))
    with pytest.raises(RuntimeError, match="older than its source"):
        build.ensure_built()
