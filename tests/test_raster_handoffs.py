"""Hand-offs through the LDS in raster.hip: every loop in which a wave's lanes read staged entries
of other lanes (``s_splat[j]``, ``s_splat[e]``) has a wave_sync() between the staging store and it,
on each path that leads there.  Such a wait cannot be missed by a result on this hardware, so the
source is read."""
import os
import re

import pytest

SRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                   "paper_2509_12138_amd", "csrc", "raster.hip")


def _body(name):
    """Text of the function `name` between its outer braces."""
    text = re.sub(r"//[^\n]*", "", open(SRC).read())
    at = text.index("{", re.search(r"\b%s\(" % name, text).end())
    depth = 0
    for i in range(at, len(text)):
        depth += {"{": 1, "}": -1}.get(text[i], 0)
        if depth == 0:
            return text[at:i + 1]
    raise AssertionError(name)


def _without_blocks_that_leave(path):
    """Drops the `if (...) { ... continue; }` blocks: a path past them did not run them."""
    out, i = [], 0
    while i < len(path):
        m = re.compile(r"\bif \(").search(path, i)
        if not m:
            out.append(path[i:])
            break
        j, depth = m.end(), 1
        while depth:
            depth += {"(": 1, ")": -1}.get(path[j], 0)
            j += 1
        k = j
        while path[k] in " \n":
            k += 1
        if path[k] == "{":
            e, depth = k, 0
            while True:
                depth += {"{": 1, "}": -1}.get(path[e], 0)
                e += 1
                if depth == 0 or e >= len(path):
                    break
            if re.search(r"continue;\s*\}$", path[k:e]):
                out.append(path[i:m.start()])
                i = e
                continue
        out.append(path[i:j])
        i = j
    return "".join(out)


@pytest.mark.parametrize("name", ["k_raster_bwd_chunked_q", "reverse_pass", "k_raster_fwd_join"])
def test_staged_entries_are_waited_for(name):
    body = _body(name)
    store = re.search(r"s_splat\[lane\] = ", body)
    assert store
    reads = [m.start() for m in re.finditer(r"= s_splat\[[ej]\]", body) if m.start() > store.end()]
    assert reads
    for r in reads:
        assert "wave_sync();" in _without_blocks_that_leave(body[store.end():r]), body[r - 200:r + 40]
