"""Every call reads the process-wide sweep setting once, so that a change by
another thread reaches it whole or not at all: the word is loaded in one place,
and each entry that depends on it asks for it once.  (What a second read could
change is the order of a pass alone, never its values, so this is read from the
source.)"""
import os
import re

from paper_2512_11473_amd import build


def _bodies(text):
    """Function name -> body, of the definitions that start in column 0."""
    got = {}
    for m in re.finditer(r"^[\w:<>\"][^\n;{}]*?(\w+)\((?:[^;{}]*)\)\s*(?:const\s*)?\{\n", text, re.MULTILINE):
        end = text.index("\n}\n", m.end())
        got.setdefault(m.group(1), "")
        got[m.group(1)] += text[m.end():end]
    return got


def test_setting_is_read_once():
    with open(os.path.join(build.CSRC, "sweep.hip")) as f:
        text = re.sub(r"//[^\n]*", "", f.read())
    bodies = _bodies(text)
    reads = {name: body.count("current_sweep_config()") for name, body in bodies.items()}
    assert text.count("g_sweep_word.load") == 1
    asks = {name for name, n in reads.items() if n}
    assert asks == {"launch_cut_fractions", "sgrid_reinitialize", "gradient_entry", "sgrid_compute_laplacian"}
    assert all(reads[name] == 1 for name in asks), reads
    # and none of them calls another that asks
    for name in asks:
        assert not any(re.search(r"\b%s\(" % other, bodies[name]) for other in asks), name
