"""Properties of the kernel sources that no output shows: what a test of
results cannot tell apart is held here."""
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2606_02218_amd", "csrc")


def _source(name):
    """A source file without its comments."""
    with open(os.path.join(CSRC, name)) as f:
        s = f.read()
    return re.sub(r"//[^\n]*|/\*.*?\*/", "", s, flags=re.S)


def test_scored_log_probabilities_use_the_library_exponential():
    """The recompute's logsumexp, in the lm head's epilogue as from written
    logits, takes expf (8.4e-8 relative at most over [-87, 0]): the fast form
    rounds x log2(e) before exponentiating, 1e-6 relative at x = -20.  A sum's
    largest terms hide most of it, so no log-probability tells the two apart."""
    for name in ("k_gemm.hip", "k_loss.hip"):
        assert not re.search(r"__expf|__builtin_amdgcn_exp2f|\bexp2f", _source(name)), name


def test_assembly_lists_the_scalar_registers_it_writes():
    """Inline assembly that sets m0 (the LDS address of a direct load) tells the
    compiler so, which keeps values of its own there (LDS and message
    instructions)."""
    found = 0
    for name in sorted(os.listdir(CSRC)):
        for m in re.finditer(r"\basm\s*(?:volatile)?\s*\((.*?)\)\s*;", _source(name), flags=re.S):
            body = m.group(1)
            if re.search(r"s_mov_b32\s+m0", body):
                found += 1
                assert '"m0"' in body.rsplit(":", 1)[1], (name, body)
    assert found


def test_restrict_pointers_of_a_call_are_distinct():
    """No call hands one pointer expression to two parameters: the kernels'
    helpers take restrict-qualified pointers, and memory that one of them
    writes may not be read through another."""
    for name in sorted(os.listdir(CSRC)):
        if not name.endswith(".hip"):
            continue
        for m in re.finditer(r"\b(\w+)(?:<[^;{}()]*>)?\(([^;{}]*)\);", _source(name)):
            args = re.findall(r"(?<![\w.>])(?:ep|a|sm|p)\.\w+(?![\w.\[(])", m.group(2))
            ptrs = [x for x in args if x.split(".")[1] in ("x", "C", "q_out", "kv_pool", "part", "norm_g", "tgt_z")]
            assert len(ptrs) == len(set(ptrs)), (name, m.group(0)[:120])
