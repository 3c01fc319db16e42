"""Host-side checks of include/eselbm_rollout.h (no GPU needed): the library
exports what it declares, the Python binding names the same functions, and
NULL arguments are refused before any device call."""
import ctypes
import pathlib
import re

ROOT = pathlib.Path(__file__).resolve().parents[1]
LIB = ROOT / "paper_2203_12946_amd" / "libeselbm.so"


def test_rollout_header_library_and_binding_agree():
    import paper_2203_12946_amd.eselbm as es
    src = re.sub(r"/\*.*?\*/", "", (ROOT / "include" / "eselbm_rollout.h").read_text(), flags=re.S)
    names = set(re.findall(r"\b(eselbm_[a-z_0-9]+)\s*\(", src))
    assert names == {"eselbm_rollout_steps", "eselbm_rollout_adjoints"} == set(es._ROLLOUT_SIGNATURES)
    lib = ctypes.CDLL(str(LIB))
    for n in names:
        # as many parameters as the binding declares
        args = re.search(n + r"\s*\(([^)]*)\)", src).group(1).split(",")
        assert hasattr(lib, n) and len(args) == len(es._ROLLOUT_SIGNATURES[n])


def test_null_arguments_are_refused():
    import paper_2203_12946_amd.eselbm as es
    assert es.lib.eselbm_rollout_steps(None, None, None, None, 1, 0.1, None, 0.0, None) == 1
    assert es.lib.eselbm_rollout_adjoints(None, None, None, 1, 0.0, None, None, 0.1, None, None) == 1
    assert b"eselbm_rollout_adjoints" in es.lib.eselbm_last_error()
