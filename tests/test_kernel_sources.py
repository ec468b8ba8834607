"""What holds for the text of every kernel."""
import glob
import os
import re

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1811_11679_amd", "csrc")


def _functions():
    """(name, is a kernel, body) of every function that is defined at the margin of a device source."""
    for path in sorted(glob.glob(os.path.join(CSRC, "*.hip")) + glob.glob(os.path.join(CSRC, "*.h"))):
        lines = open(path).read().split("\n")
        for i, line in enumerate(lines):
            if line != "{":
                continue
            j = i
            while j > 0 and lines[j - 1] and not lines[j - 1].startswith(("}", "//", "#")):
                j -= 1
            head = " ".join(lines[j:i])
            names = re.findall(r"(\w+)\(", re.sub(r"__\w+__\s*\((?:[^()]|\([^()]*\))*\)", "", head))
            if names and "__" in head:
                yield names[0], "__global__" in head, "\n".join(lines[i:lines.index("}", i)])


def test_blocks_agree_on_an_error():
    """A kernel with barriers whose own launch may set an error bit asks once per
    block whether one is set: waves that looked for themselves could disagree
    while another block sets it."""
    sets = r"atomicOr\(&[^;]*err,"
    bodies = {name: (kernel, body) for name, kernel, body in _functions()}
    helpers = [n for n, (kernel, body) in bodies.items() if not kernel and re.search(sets, body)]
    assert "det_update" in helpers
    seen = []
    for name, (kernel, body) in bodies.items():
        raises = re.search(sets, body) or any(re.search(rf"\b{h}\(", body) for h in helpers)
        if not kernel or "__syncthreads" not in body or not raises:
            continue
        seen.append(name)
        assert "block_stops(c)" in body, name
        assert not re.search(r"if \(c->err", body), name
    assert {"k_spawn", "k_collapse", "k_merge", "k_move", "k_ccmc_clusters", "k_det_project_split"} <= set(seen), seen
