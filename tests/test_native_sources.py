"""CPU: whoever builds the library's sources by a list of their own links the whole library.

The sanitizer driver (tests/native/build_sanitized.sh) names the translation units itself.  They have to be
build.py's, and every source file under csrc has to be one of them or be included by one.
"""
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1609_08146_amd", "csrc")


def test_sanitizer_driver_names_the_librarys_translation_units():
    from paper_1609_08146_amd import build
    text = open(os.path.join(ROOT, "tests", "native", "build_sanitized.sh")).read()
    named = set(re.findall(r"\bsc_[a-z_]+\.(?:hip|cpp)\b", text))
    linked = {os.path.basename(o) for o in re.findall(r'"\$OUT"/(sc_[a-z_]+)\.o', text.split(" -o \"$OUT/abi_$SAN\" ")[-1])}
    assert named == set(build.SOURCES)
    assert linked == {os.path.splitext(s)[0] for s in build.SOURCES}


def test_every_source_belongs_to_a_translation_unit():
    from paper_1609_08146_amd import build
    reached, todo = set(), list(build.SOURCES)
    while todo:
        name = todo.pop()
        if name in reached:
            continue
        reached.add(name)
        with open(os.path.join(CSRC, name)) as fh:
            todo += re.findall(r'^#include "(sc_[a-z_]+\.(?:hip|cpp))"', fh.read(), re.M)
    alone = {"valu_rates.hip"}   # a program of its own (instruction rates), not part of the library
    assert reached == {f for f in os.listdir(CSRC) if f.endswith((".hip", ".cpp"))} - alone
