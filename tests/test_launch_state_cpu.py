"""State that launchers keep between calls: threads share it, and what it says of one GPU need not hold for the next."""
import glob
import os
import re

import paper_2604_23108_amd as M

CSRC = os.path.join(os.path.dirname(M.lib_path()), "csrc")


def test_launchers_keep_only_atomic_state():
    for path in sorted(glob.glob(os.path.join(CSRC, "*.hip")) + glob.glob(os.path.join(CSRC, "*.h"))):
        text = re.sub(r"//[^\n]*", "", open(path).read())
        kept = re.findall(r"^[ \t]+static (?!constexpr|const |std::atomic)[\w:<> ]+?[*& ]\w+(?:\[\w*\])?\s*(?:=|\{|;)", text, flags=re.M)
        assert not kept, f"{os.path.basename(path)}: {kept}"


def test_large_dynamic_lds_is_allowed_per_gpu():
    """Kernels with more than 64 KB of dynamic LDS have to be allowed to on every GPU: one helper keeps a bit for each."""
    for path in glob.glob(os.path.join(CSRC, "*.hip")):
        assert "hipFuncSetAttribute" not in open(path).read(), os.path.basename(path)
