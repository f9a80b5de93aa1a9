"""The constants of the fp64 normals in the source are those that their
generator makes."""
import importlib.util
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_header_holds_what_the_generator_makes():
    spec = importlib.util.spec_from_file_location(
        "make_normal_tables", os.path.join(ROOT, "tests", "golden", "make_normal_tables.py"))
    gen = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(gen)
    src = open(os.path.join(ROOT, "paper_1505_00965_amd", "csrc", "normal64.hpp")).read()
    num = r"-?0x[0-9a-f.]+p[-+]?\d+|-?\d+\.\d+"

    def numbers(text):
        return [float.fromhex(t) if "0x" in t else float(t) for t in re.findall(num, text)]

    for name, want in gen.constants().items():
        text = re.search(r"\b%s(?:\[[^=]*)? = ([^;]*?)(;|, k)" % name, src, re.S).group(1)
        flat = [x for row in want for x in (row if isinstance(row, tuple) else [row])] if isinstance(want, list) else [want]
        assert numbers(text) == flat, name
