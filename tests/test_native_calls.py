"""The native calls of a serving loop (csrc/pycalls.cpp) against the ctypes functions that they stand in for: the same plans, the same
errors, for arguments that they read themselves and for those that they hand on."""
import ctypes as C

import pytest

import paper_2407_21418_amd as ft
from paper_2407_21418_amd import binding

NATIVE = {n: getattr(binding, n) for n in ("ft_plan_cached", "ft_launch", "ft_launch_epilogue")}


def slow(name):
    """The ctypes function: what the native one calls for keywords."""
    lib = binding.lib()
    if name == "ft_plan_cached":
        def f(op, s, shape, flags=0):
            out = C.c_void_p()
            binding._check(lib.ft_plan_cached(op.ptr, s.ptr, C.byref(shape), flags, C.byref(out)), name)
            return binding.CachedPlan(out.value, s)
    elif name == "ft_launch":
        def f(p, A, B, Cptr, stream=0):
            binding._check(lib.ft_launch(p.ptr, A, B, Cptr, stream), name)
    else:
        def f(p, A, B, Cptr, bias, stream=0):
            binding._check(lib.ft_launch_epilogue(p.ptr, A, B, Cptr, bias or None, stream), name)
    return f


def outcome(f, *a, **kw):
    try:
        r = f(*a, **kw)
        return ("plan", r.ptr, r._owner) if isinstance(r, binding.CachedPlan) else ("value", r)
    except Exception as e:
        return (type(e), getattr(e, "status", None))


@pytest.fixture(scope="module")
def op_set():
    op = ft.ft_op_register(ft.ft_op_desc(kind=ft.FT_OP_MATMUL, n=768, k=768, m_lo=1, m_hi=8192))
    return op, ft.ft_ukernels_derive(op)


def test_the_built_calls_are_in_use():
    assert binding._pycalls is not None and all(type(f).__name__ == "builtin_function_or_method" for f in NATIVE.values())
    assert all(getattr(ft, n) is f for n, f in NATIVE.items())


def test_plans(op_set):
    op, s = op_set
    host = ft.FT_PLAN_HOST_ONLY
    for m in (1, 77, 8192, 77):
        a, b = outcome(NATIVE["ft_plan_cached"], op, s, ft.ft_shape(m=m), host), outcome(slow("ft_plan_cached"), op, s, ft.ft_shape(m=m), host)
        assert a == b and a[0] == "plan" and a[1] and a[2] is s
    assert outcome(NATIVE["ft_plan_cached"], op, s, shape=ft.ft_shape(m=77), flags=host) == outcome(slow("ft_plan_cached"), op, s, ft.ft_shape(m=77), host)
    closed = binding.UkSet(None)
    odd = ft.ft_shape(m=77)
    odd.struct_size = 4
    for args in ((op, s, ft.ft_shape(m=0)), (op, s, ft.ft_shape(m=8193)), (op, closed, ft.ft_shape(m=77)), (op, s, odd), (op, s, None), (op, s, 3), (None, s, ft.ft_shape(m=1)),
                 (op, s, ft.ft_hw_model()), (op, s), (op, s, ft.ft_shape(m=1), 16, 5)):
        a = outcome(NATIVE["ft_plan_cached"], *args)
        assert a == outcome(slow("ft_plan_cached"), *args) and isinstance(a[0], type), args


@pytest.mark.parametrize("name,more", [("ft_launch", ()), ("ft_launch_epilogue", (0,))])
def test_launch_errors(op_set, name, more):
    """Every call here is turned down before anything reaches a GPU: the plan is host-only, or there is none."""
    op, s = op_set
    plan = ft.ft_plan_create(op, s, ft.ft_shape(m=77), ft.FT_PLAN_HOST_ONLY)
    none = binding.Plan(None)
    for args in ((plan, 16, 16, 16), (plan, 16, 16, 16, 0), (plan, 0, 16, 16), (plan, None, 16, 16), (none, 16, 16, 16), (plan, C.c_void_p(16), 16, 16), (plan, True, 16, 16),
                 (plan, 16, 2 ** 64 + 16, 16), (plan, -16, 16, 16), (plan, 16.0, 16, 16), (plan, "x", 16, 16), (None, 16, 16, 16), (plan, 16, 16)):
        args = args[:4] + more + args[4:]
        a = outcome(NATIVE[name], *args)
        assert a == outcome(slow(name), *args) and isinstance(a[0], type), args
    assert outcome(NATIVE[name], plan, A=16, B=16, Cptr=16, **({"bias": 0} if more else {})) == (ft.FtError, ft.FT_ERR_INVALID_ARG)


def test_structures_take_their_fields():
    sh = ft.ft_shape(m=77, batch=2)
    assert (sh.struct_size, sh.m, sh.batch, sh.n) == (C.sizeof(ft.ft_shape), 77, 2, 0)
    assert ft.ft_shape(struct_size=4).struct_size == 4 and ft.ft_shape().struct_size == C.sizeof(ft.ft_shape)
