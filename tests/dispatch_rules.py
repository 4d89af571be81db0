"""The library's own rules, which say what kernel a call takes (host functions of libzeda.so, plain C++ symbols), so that a test can
hold a case to the path that it is there for."""
import ctypes

from paper_2605_18643_amd import zeda


def _rule(name, res):
    f = getattr(zeda.lib(), f"_ZN4zeda{len(name)}{name}EPK15zeda_layer_desc")
    f.argtypes, f.restype = [ctypes.POINTER(zeda.LayerDesc)], res
    return lambda d: f(ctypes.byref(d))


few_blocks = _rule("ffn_few_blocks", ctypes.c_int)         # 16-row token blocks of the few-row kernel's workgroups, 0: not that kernel
gateup_places = _rule("gateup_places", ctypes.c_bool)      # a whole-layer call places in the gate/up kernel
gateup_selects = _rule("gateup_selects", ctypes.c_bool)    # ... and selects there
route_splits = _rule("route_splits", ctypes.c_bool)        # the router is two kernels
route_places = _rule("route_places", ctypes.c_bool)        # the second one can place


def whole_layer_places(d):
    """Who places in a whole-layer call."""
    if gateup_places(d):
        return "gateup"
    return "router" if route_places(d) else "launch"
