"""What can be said about the kernel sources without a GPU."""
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2512_17077_amd", "csrc")

# preprocessor names the sources may test: the checked build and one size
KNOWN = {"DLLM_CHECK_PRECONDITIONS", "DLLM_PACK_INFLIGHT", "DLLM_PRECONDITION_RULES_H", "DLLM_SCORE_RULES_H",
         "__HIPCC__"}


def test_no_undocumented_switches():
    found = set()
    for name in os.listdir(CSRC):
        if name.endswith((".hip", ".h", ".inc")):
            for line in open(os.path.join(CSRC, name)):
                if re.match(r"\s*#\s*(if|ifdef|ifndef|elif)\b", line):
                    found |= set(re.findall(r"\b[A-Z_][A-Z0-9_]{2,}\b", line))
    assert found <= KNOWN, f"switches nobody documents: {sorted(found - KNOWN)}"
