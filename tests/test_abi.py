"""The C-ABI library loads and exports every entry point include/libecc.h
declares; host-only validation returns the documented status codes.  No GPU
call is made here."""
import os
import re

import numpy as np
import pytest

from paper_2203_17063_amd import capi as E

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def header_functions():
    text = open(os.path.join(ROOT, "include", "libecc.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)        # drop comments
    names = re.findall(r"^[A-Za-z_][\w \*]*?\b(ecc_\w+)\s*\(", text, flags=re.M)
    return sorted(set(names))


def exported_symbols():
    import subprocess
    out = subprocess.run(["nm", "-D", "--defined-only", E.LIB_PATH], capture_output=True,
                         text=True, check=True).stdout
    return sorted(l.split()[-1] for l in out.splitlines() if " T ecc_" in l)


def test_library_loads_and_exports_header():
    E.lib()
    decl = header_functions()
    assert len(decl) >= 19
    exp = exported_symbols()
    assert decl == exp
    assert sorted(E.EXPORTED) == decl          # the binding covers every entry point
    assert E.ecc_abi_version() == 3


def header_constants():
    """Every integer constant the header defines: #define lines and the
    status enum."""
    text = open(os.path.join(ROOT, "include", "libecc.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    consts = {m.group(1): int(m.group(2), 0)
              for m in re.finditer(r"^#define\s+(ECC_\w+)\s+((?:0x)?[0-9a-fA-F]+)\s*$", text,
                                   flags=re.M)}
    consts.update({m.group(1): int(m.group(2))
                   for m in re.finditer(r"\b(ECC_(?:OK|ERR_\w+))\s*=\s*(\d+)", text)})
    return consts


def test_binding_constants_match_header():
    consts = header_constants()
    assert len(consts) >= 24
    for name, value in consts.items():
        assert getattr(E, name) == value, name


def test_status_strings():
    for code, name in E.STATUS_NAMES.items():
        assert E.lib().ecc_status_string(code).decode() == name


@pytest.mark.parametrize("P,counts,displs,S,expect", [
    (0, None, None, 0, E.ECC_ERR_ARG),                       # P < 1
    (3, None, None, -1, E.ECC_ERR_ARG),                      # negative staleness
    (3, None, None, 0, E.ECC_OK),                            # allreduce-only plan
    (3, [1, 2, 3], None, 0, E.ECC_ERR_ARG),                  # counts without displs
    (3, [1, -2, 3], [0, 1, 3], 0, E.ECC_ERR_ARG),            # negative count
    (3, [1, 2, 3], [0, -1, 3], 0, E.ECC_ERR_ARG),            # negative displacement
    (3, [2, 2, 2], [0, 1, 4], 0, E.ECC_ERR_OVERLAP),         # overlap
    (3, [2, 0, 2], [0, 1, 2], 0, E.ECC_OK),                  # empty block may sit anywhere
    (3, [2, 2, 2], [4, 0, 10], 0, E.ECC_OK),                 # unsorted with gaps
    (2, [1, 1], [0, 1 << 40], 0, E.ECC_ERR_RANGE),           # beyond 2^40
    (4, [5, 5, 5, 5], [0, 5, 10, 15], E.ECC_UNBOUNDED, E.ECC_OK),
])
def test_plan_validate(P, counts, displs, S, expect):
    assert E.ecc_plan_validate(P, counts, displs, S) == expect
    if expect != E.ECC_OK:
        assert E.ecc_last_error() != ""


def test_null_handles_are_rejected_without_device():
    L = E.lib()
    assert L.ecc_plan_reset(None) == E.ECC_ERR_ARG
    assert L.ecc_plan_destroy(None) == E.ECC_OK
    assert L.ecc_matrix_destroy(None) == E.ECC_OK
    assert L.ecc_partials_size(None) == 0
    assert L.ecc_allgatherv_assemble(None, None, None, None, None, None) == E.ECC_ERR_ARG
    assert L.ecc_residual(None, None, 1, 2, None, None) == E.ECC_ERR_ARG
    assert L.ecc_matrix_layout(None, None, None) == E.ECC_ERR_ARG


def test_product_path_does_not_touch_oracle():
    """The package and the HIP sources never import, link or call the oracle."""
    pkg = os.path.join(ROOT, "paper_2203_17063_amd")
    for dirpath, _, files in os.walk(pkg):
        for f in files:
            if f.endswith((".py", ".hip", ".h", ".cpp")):
                text = open(os.path.join(dirpath, f)).read()
                for bad in ("import oracle", "from oracle", "liboracle", "orc_"):
                    assert bad not in text, (f, bad)


@pytest.mark.parametrize("P,m,slack,expect", [
    (0, 16, 0, E.ECC_ERR_ARG),                        # P < 1
    (3, 16, 0, E.ECC_ERR_ARG),                        # not a power of two
    (8192, 16, 0, E.ECC_ERR_ARG),                     # beyond 4096 processes
    (4, -1, 0, E.ECC_ERR_ARG),                        # negative length
    (4, 16, -1, E.ECC_ERR_ARG),                       # negative slack
    (4, (1 << 40) // 8 + 1, 0, E.ECC_ERR_RANGE),      # slots beyond 2^40 elements
    (1, 0x7fffffff * 64 + 1, 0, E.ECC_ERR_RANGE),     # beyond the grid's 64 elements per workgroup
])
def test_hypercube_create_checks_without_device(P, m, slack, expect):
    """Argument and range checks return before any device call."""
    with pytest.raises(E.EccError) as err:
        E.ecc_hypercube_create(P, m, slack)
    assert err.value.status == expect


def test_allreduce_shapes():
    """The partial allreduce's launch over ranks, lengths and whether the
    contributions are held in their slots: no access is wider than the vector,
    and the summing threads cover it."""
    lengths = {0, 1, 2, 3, 600}
    for e in (4096, 65536, 1 << 19, 200 * 4096, 200 * 8192, 200 * 16384, 1 << 32):
        lengths |= {e - 1, e, e + 1}
    for P in (1, 2, 15, 16, 17, 256, 1024, 1025, 5000, (1 << 24) - 1):
        for m in sorted(lengths):
            for held in (False, True):
                groups, threads, width = E.ecc_allreduce_shape(P, m, held)
                assert threads % 64 == 0 and width in (1, 2) and groups >= 1
                assert m == 0 or width <= m, (P, m, held)
                assert m == 0 or groups >= 2, (P, m, held)
    assert E.lib().ecc_allreduce_shape(0, 1, 0, None, None, None) == E.ECC_ERR_ARG


@pytest.mark.parametrize("held", [False, True])
@pytest.mark.parametrize("P", [1, 2, 15, 16, 17, 1024, 1025])
def test_allreduce_longest_vectors(P, held):
    """A launch holds fewer than 2^32 threads: vectors of up to nearly 2^36
    elements (one element per 16 in a thread) fit one whatever the ranks."""
    for m in (1 << 31, (1 << 32) - 1, 1 << 32, (1 << 33) - 1, 1 << 33, (1 << 33) + 1, 1 << 34,
              (1 << 35) + 3, (1 << 36) - (1 << 15)):
        groups, threads, _ = E.ecc_allreduce_shape(P, m, held)
        assert groups * threads < 1 << 32, (P, m, held)


def test_allreduce_wide_chunks_run_together():
    """Chunks of 16 elements per thread below the widest are taken only while
    the device's 256 CUs hold all of their workgroups, one each."""
    for P in (16, 48, 256, 2000):
        for m in range(600001, 5000000, 99991):
            groups, threads, _ = E.ecc_allreduce_shape(P, m)
            if threads < 1024 and m > 8 * threads * (groups - 1):
                assert 100 <= groups - 1 <= 256, (P, m, groups)


def test_allreduce_held_range():
    """Contributions held in their slots have a shape of their own between
    256 MiB and 1 GiB of them only."""
    for P in (16, 24, 64, 256, 2000):
        for m in (70001, 150001, 400000, 1700001, 3520000, 4194304, 8000001):
            own = E.ecc_allreduce_shape(P, m, True) != E.ecc_allreduce_shape(P, m, False)
            assert own == (256 << 20 < 8 * P * m < 1 << 30), (P, m)
