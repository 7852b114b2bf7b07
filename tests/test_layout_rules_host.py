"""The digest that tells whether the committed traffic figures still hold
covers the rules that choose what the kernels run on."""

import os

from paper_2306_04322_amd import build as B


def test_digest_covers_the_layout_rules():
    for rule in ("tiled_layout(int", "one_pass_strided(int", "row_major_spectra(int"):
        files = [n for n in sorted(os.listdir(B.CSRC)) if rule in open(os.path.join(B.CSRC, n)).read()]
        assert files and set(files) <= set(B.FS_F32_KERNEL_SOURCES), (rule, files)
