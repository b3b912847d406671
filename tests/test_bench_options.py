"""Every mode of the benchmark defines the options that it reads."""

import ast
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_every_mode_defines_the_options_it_reads():
    with open(os.path.join(ROOT, "bench.py")) as f:
        src = f.read()
    parsed = {m.replace("-", "_") for m in re.findall(r'add_argument\("--([\w-]+)"', src)}
    funcs = {n.name: n for n in ast.parse(src).body if isinstance(n, ast.FunctionDef)}
    options, own, calls = {}, {}, {}
    for name, fn in funcs.items():
        attrs = [n for n in ast.walk(fn) if isinstance(n, ast.Attribute)
                 and isinstance(n.value, ast.Name) and n.value.id == "args"]
        options[name] = {n.attr for n in attrs if isinstance(n.ctx, ast.Load)}
        own[name] = {n.attr for n in attrs if isinstance(n.ctx, ast.Store)}
        calls[name] = {n.func.id for n in ast.walk(fn) if isinstance(n, ast.Call)
                       and isinstance(n.func, ast.Name) and n.func.id in funcs}
    entries = [n for n in funcs if n.endswith("_mode")] + ["main"]
    assert "farfield_mode" in entries and "tol" in parsed
    for entry in entries:
        reach, todo = set(), [entry]
        while todo:
            f = todo.pop()
            if f not in reach:
                reach.add(f)
                todo += calls[f]
        read = set().union(*(options[f] for f in reach))
        missing = read - parsed - set().union(*(own[f] for f in reach))
        assert not missing, (entry, missing)
