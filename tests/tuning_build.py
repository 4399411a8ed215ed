"""The tuning build of the library (-DAWQ_TUNING_KNOBS) in the place of the product for a few calls, with some of its
overrides set.  The ones used this way are read at every call; those that are read once per process need a
process of their own."""
import contextlib
import os

import paper_2306_00978_amd as awq

_loaded = []


def _library():
    if not _loaded:
        product, awq._lib = awq.load(), None
        before = os.environ.get("AWQ_MI355X_LIBRARY")
        os.environ["AWQ_MI355X_LIBRARY"] = awq.LIB_PATH.replace(".so", "_knobs.so")
        try:
            _loaded.append(awq.load())
        finally:
            awq._lib = product
            if before is None:
                del os.environ["AWQ_MI355X_LIBRARY"]
            else:
                os.environ["AWQ_MI355X_LIBRARY"] = before
    return _loaded[0]


@contextlib.contextmanager
def tuning_build(**overrides):
    """Without an override that is not None: the product."""
    overrides = {k: str(v) for k, v in overrides.items() if v is not None}
    if not overrides:
        yield
        return
    library, product = _library(), awq.load()
    os.environ.update(overrides)
    awq._lib = library
    try:
        yield
    finally:
        awq._lib = product
        for name in overrides:
            del os.environ[name]
