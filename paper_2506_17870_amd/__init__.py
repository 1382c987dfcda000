"""NestQuant nested-integer hot path for AMD MI355X (gfx950): hand-written HIP kernels
behind a C ABI (include/nq.h) with a thin binding.  PyTorch is used only for device
memory and streams.

The binding (and with it libnq.so) is loaded on first use of any attribute, so that
`python -m paper_2506_17870_amd.build` can run before the library exists; using the package
without a built library raises ImportError -- there is no fallback path.
"""
import importlib

__all__ = ["binding", "build", "inputs"]
_copied = {}                           # what the package holds of the binding's attributes


def __getattr__(name):
    if name in ("build", "inputs", "binding"):
        return importlib.import_module(f"{__name__}.{name}")
    binding = importlib.import_module(f"{__name__}.binding")
    try:
        value = getattr(binding, name)
    except AttributeError:
        raise AttributeError(f"module {__name__!r} has no attribute {name!r}") from None
    globals()[name] = _copied[name] = value        # the next access does not come here (3.5 us, as much as a layer's whole call)
    return value


def _forget(*names):
    """Called by the binding when attributes of its own are replaced: the next access through the package asks it again."""
    for name in names or list(_copied):
        value = _copied.pop(name, _copied)
        if value is not _copied and globals().get(name, _copied) is value:       # (the caller may have put something else here)
            globals().pop(name, None)
