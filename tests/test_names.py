"""A test function that is defined twice in a module replaces the first one silently: every name is defined once."""
import ast
import glob
import os

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.mark.parametrize("path", sorted(glob.glob(os.path.join(HERE, "test_*.py"))), ids=os.path.basename)
def test_names_are_defined_once(path):
    with open(path) as f:
        names = [n.name for n in ast.parse(f.read()).body if isinstance(n, ast.FunctionDef)]
    assert sorted(names) == sorted(set(names))
