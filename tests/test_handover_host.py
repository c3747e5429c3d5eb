"""CPU source check of the sums that workgroups hand to the last of them
(reduce.hip, paths.hip): without fences the handover holds only while the
shared words are accessed by agent-scope atomics alone and the wave waits for
them before it takes its ticket."""
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1909_10690_amd", "csrc")


def body(name, kernel):
    text = open(os.path.join(CSRC, name)).read()
    start = text.index(kernel + "(")
    text = text[start:text.index("\n}\n", start)]
    return re.sub(r"//[^\n]*", "", text)


def test_reduction_handover():
    k = body("reduce.hip", "void mi_reduce_kernel")
    # every use of the slices' sums and of the count is an agent-scope atomic (part is formed from L.part once)
    for use in re.findall(r"[^;{}]*\bpart\b[^;{}]*;", k):
        assert "__hip_atomic_" in use and "__HIP_MEMORY_SCOPE_AGENT" in use or "L.part" in use, use
    for use in re.findall(r"[^;{}]*L\.count\[t\][^;{}]*;", k):
        assert "__hip_atomic_" in use and "__HIP_MEMORY_SCOPE_AGENT" in use, use
    store, wait, ticket = (k.index(s) for s in ("__hip_atomic_store(part", "s_waitcnt vmcnt(0)", "__hip_atomic_fetch_add(&L.count[t]"))
    assert store < wait < ticket < k.index("__hip_atomic_load(part")


def test_path_figures_handover():
    k = body("paths.hip", "void path_sink_kernel")
    done = k.index("gridDim.x - 1) return;")
    for use in re.findall(r"[^;{}]*\bst\[[^;{}]*;", k):
        assert "__hip_atomic_" in use and "__HIP_MEMORY_SCOPE_AGENT" in use, use
    assert "stats[" not in k[:done]  # plain accesses only by the last workgroup, after all others
    assert k.index("__hip_atomic_fetch_min(&st[3]") < k.index("s_waitcnt vmcnt(0)") < k.index("__hip_atomic_fetch_add(&st[1]") < done
