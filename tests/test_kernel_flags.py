"""The workgroup-local kernels end early on words that say that the call is
over. A kernel whose workgroups may set such a word must not test it wave by
wave: between two waves' reads another workgroup can set it, and the waves that
stay work on LDS that the others never wrote. Such a kernel reads the words
through call_ended (one thread, then a barrier). Checked on the sources."""
import os
import re

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1501_04706_amd", "csrc")
WORDS = ("err", "left", "stop")
FILES = [os.path.join(CSRC, f) for f in ("sqh_local.hip", "sqh_ring.hpp", "sqh_sieve_large.hpp", "sqh_subset.hpp",
                                         "sqh_sieve.hpp", "sqh_dense.hpp", "sqh_solve.hpp")]


def functions():
    """name -> (is a kernel, body) of every device function of the files."""
    out = {}
    for path in FILES:
        text = re.sub(r"//[^\n]*", "", open(path).read())
        text = re.sub(r"__launch_bounds__\([^()]*\)", "", text)
        for m in re.finditer(r"(__global__|__device__)[^;{}()]*?\b(\w+)\s*\([^;{}]*?\)\s*(?:const)?\s*\{", text):
            depth, i = 1, m.end()
            while depth:
                depth += {"{": 1, "}": -1}.get(text[i], 0)
                i += 1
            out[m.group(2)] = (m.group(1) == "__global__", text[m.end():i])
    return out


FUNCS = functions()


def reach(name, seen=None):
    seen = set() if seen is None else seen
    if name not in seen:
        seen.add(name)
        for callee in set(re.findall(r"\b(\w+)\s*(?:<[^;(){}]*>)?\s*\(", FUNCS[name][1])) & set(FUNCS):
            reach(callee, seen)
    return seen


def writes(body, word):
    return bool(re.search(r"atomicOr\(&(?:a\.)?ctl->%s\b" % word, body) or re.search(r"\bctl->%s\s*=[^=]" % word, body))


def bare_reads(body, word):
    body = re.sub(r"(atomicOr|call_ended|__hip_atomic_load)\([^;]*?;", ";", body)
    return [m for m in re.finditer(r"\bctl->%s\b(?!\s*=[^=])" % word, body)]


def test_kernels_are_found():
    kernels = {n for n, (k, _) in FUNCS.items() if k}
    assert {"k_batch_big", "k_batch_small", "k_ring_cut", "k_ring_pocket", "k_sieve", "k_rest", "k_pre_keep"} <= kernels
    assert "put_hull" in reach("k_batch_small") and writes(FUNCS["put_hull"][1], "err")


@pytest.mark.parametrize("kernel", sorted(n for n, (k, _) in FUNCS.items() if k))
@pytest.mark.parametrize("word", WORDS)
def test_no_kernel_tests_a_word_it_sets(kernel, word):
    bodies = [FUNCS[f][1] for f in reach(kernel)]
    if any(writes(b, word) for b in bodies):
        assert not any(bare_reads(b, word) for b in bodies)
