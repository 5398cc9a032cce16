"""A second definition of a name in a test file replaces the first one, whose cases then never run."""
import ast
import glob
import os

import pytest

FILES = sorted(glob.glob(os.path.join(os.path.dirname(os.path.abspath(__file__)), "*.py")))


@pytest.mark.parametrize("path", FILES, ids=os.path.basename)
def test_no_name_is_defined_twice(path):
    with open(path) as f:
        tree = ast.parse(f.read())
    for scope in [tree] + [n for n in ast.walk(tree) if isinstance(n, ast.ClassDef)]:
        names = [n.name for n in scope.body if isinstance(n, (ast.FunctionDef, ast.AsyncFunctionDef, ast.ClassDef))]
        assert sorted(names) == sorted(set(names)), sorted(n for n in set(names) if names.count(n) > 1)
