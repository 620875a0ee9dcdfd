"""Every table of fitness kernel instances is compiled with the unroll limit that its weight
source needs (no GPU, no compiler): tables are found by what they hold, not by their file's
name, and an entry of a kind that is not known here fails."""
import os
import re

from paper_2501_03944_amd import build
from test_build_config import CSRC, FIXED, WL_ARG

STAGED = {"FIT_ENTRY_SPLIT"}      # weights always staged in LDS


def _tables():
    for name in sorted(f for f in os.listdir(CSRC) if f.endswith(".hip")):
        text = open(os.path.join(CSRC, name)).read()
        if "kEntries[] = {" in text:
            body = text[text.index("kEntries[] = {"):]
            yield name, re.sub(r"//[^\n]*", "", body[:body.index("};")])


def _global(body):
    """Whether each entry reads its weights from global memory."""
    out = []
    for m in re.finditer(r"\b(FIT_\w+)\s*\(([^)]*)\)", body):
        macro, args = m.group(1), [a.strip() for a in m.group(2).split(",")]
        if macro in STAGED:
            out.append(False)
            continue
        assert macro in FIXED or macro in WL_ARG, macro
        wl = FIXED[macro] if macro in FIXED else args[WL_ARG[macro]]
        assert wl in ("true", "false"), (macro, args)
        out.append(wl == "false")
    assert len(out) == len(re.findall(r"\bFIT_\w+", body)), body
    return out


def test_every_table_has_its_unroll_limit():
    tables = dict(_tables())
    assert {"lds_any.hip", "split_any.hip", "split_relu.hip"} <= set(tables)
    for name, body in tables.items():
        entries = _global(body)
        assert entries, name
        assert all(entries) == (name in build.GLOBAL_WEIGHT_SOURCES), name
    assert set(build.GLOBAL_WEIGHT_SOURCES) <= set(tables) <= set(build.SOURCES)


def test_tables_are_what_the_host_selects_from():
    """Each table's accessor is listed once where plans are made."""
    host = open(os.path.join(CSRC, "fitness.hip")).read()
    listed = re.findall(r"\btable_\w+", host[host.index("kTables[])"):host.index("};", host.index("kTables[])"))])
    for name, _ in _tables():
        defined = re.findall(r"KernelEntry \*(table_\w+)\(", open(os.path.join(CSRC, name)).read())
        assert defined and all(listed.count(t) == 1 for t in defined), (name, defined)
