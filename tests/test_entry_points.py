"""C entry points turn every C++ exception into a status: one that escapes a C
caller's frame ends the process."""
import glob
import os
import re

from tests.conftest import ROOT

SOURCES = sorted(glob.glob(os.path.join(ROOT, "paper_2512_07311_amd", "csrc", "*.hip")) +
                 glob.glob(os.path.join(ROOT, "paper_2512_07311_amd", "csrc", "*.cpp")))


def _handlers(text):
    """What each chain of catch clauses after a try block's end catches."""
    for m in re.finditer(r"\}\s*\\?\s*catch \(const rcs::Error& e\)", text):
        chain, at = ["rcs::Error"], m.end()
        while True:
            body = re.compile(r"\s*\\?\s*\{(?:[^{}]|\{[^{}]*\})*\}\s*\\?\s*catch \(([^)]*)\)").match(text, at)
            if not body:
                break
            chain.append(body.group(1))
            at = body.end()
        yield chain


def test_every_entry_point_catches_all_exceptions():
    n = 0
    for path in SOURCES:
        text = open(path).read()
        if 'extern "C"' not in text:
            continue
        for chain in _handlers(text[text.index('extern "C"'):] + text[:text.index('extern "C"')]):
            assert chain[-1] == "const std::exception& e", (os.path.basename(path), chain)
            n += 1
        # every entry point has such a block
        for name, body in re.findall(r"^rcs_status (rcs_\w+)\([^)]*\) \{\n(.*?)^\}", text, re.S | re.M):
            assert re.match(r"\s*(try \{|RCS_API_BEGIN|return rcs_)", body), name
    assert n >= 9
