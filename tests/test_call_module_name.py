"""The module with the hot calls carries the interpreter's ABI tag: one built for another version is not found, instead of being
loaded as it is."""
import importlib.machinery
import os
import sysconfig

from paper_1901_01544_amd import build, iwp


def test_tagged():
    iwp.load()
    path = iwp._hot().__file__
    assert os.path.basename(path) == "_call" + sysconfig.get_config_var("EXT_SUFFIX")
    assert os.path.samefile(path, build.CALL)
    tag = importlib.machinery.EXTENSION_SUFFIXES[0]
    assert tag not in (".so", ".abi3.so") and path.endswith(tag)
    assert not os.path.exists(os.path.join(os.path.dirname(path), "_call.so"))
