"""The lines between the launch forms, on the CPU: the rules are host code of their own headers, built with g++ and asked for
the sizes on both sides of each line, as timed on the card (figures beside the rules), and for what every form must cover."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "..", "paper_2606_21868_amd", "csrc")

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("rules") / "rules_check")
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-I", CSRC, os.path.join(HERE, "native", "rules_check.cpp"), "-o", exe],
                   check=True, timeout=120)

    def run(questions):
        args = [str(a) for q in questions for a in q]
        r = subprocess.run([exe, *args], capture_output=True, text=True, timeout=60)
        assert r.returncode == 0
        return [tuple(int(v) for v in line.split()) for line in r.stdout.splitlines()]
    return run


# tokens, experts, d_model, and whether small workgroups are the faster form there
@pytest.mark.parametrize("T,N,d,fine", [
    (9, 256, 7168, True), (700, 256, 7168, True), (800, 256, 7168, False), (1024, 256, 7168, False),
    (1040, 256, 7168, False), (1984, 256, 7168, False), (2500, 256, 7168, False),
    (600, 192, 4096, True), (700, 192, 4096, False), (1900, 192, 4096, False),
    (37, 128, 2048, True), (1024, 128, 2048, True), (1040, 128, 2048, False), (1900, 128, 2048, False), (2048, 128, 2048, False),
    (301, 64, 7168, True), (1024, 64, 7168, True), (1040, 64, 7168, False), (2500, 64, 7168, False), (203, 60, 1472, True)])
def test_router_form(ask, T, N, d, fine):
    slices, steps, tb, groups, rb = ask([("router", T, N, d)])[0]
    assert (tb < 4) == fine


def test_router_forms_cover_every_row_and_column(ask):
    q = [("router", T, N, d) for T in (9, 16, 17, 64, 65, 500, 1024, 1025, 2048, 2049, 5000) for N in (1, 16, 60, 64, 65, 130, 192, 256)
         for d in (16, 64, 320, 1472, 2048, 7168)]
    for (_, T, N, d), (slices, steps, tb, groups, rb) in zip(q, ask(q)):
        assert 1 <= slices <= 8 and (slices - 1) * steps < d // 16 <= slices * steps
        assert tb in (1, 2, 4) and groups * rb * 64 >= N > (groups * rb - 1) * 64
        assert (rb == 1 and groups >= 1) if tb < 4 else groups == 1


# widths, bytes of a weight, tokens, and whether streaming whole rows is the faster form there
@pytest.mark.parametrize("d,I,elem,T,stream", [
    (2048, 768, 2, 1, False), (2048, 768, 2, 2, True), (2048, 768, 2, 15, True), (2048, 768, 2, 16, False), (7168, 2048, 1, 1, True),
    (4096, 14336, 2, 4, True), (5120, 8192, 2, 4, True), (1472, 704, 2, 8, True), (1024, 1536, 2, 8, True), (1536, 768, 2, 8, True),
    (256, 128, 2, 8, False), (512, 512, 2, 8, False), (512, 4096, 2, 8, False), (1024, 1024, 2, 8, False), (960, 960, 2, 8, False),
    (768, 1024, 2, 8, False), (2048, 256, 2, 8, False), (128, 320, 2, 8, False), (384, 768, 2, 3, False), (320, 192, 2, 8, False),
    (2048, 768, 1, 2, True), (2944, 768, 1, 1, True), (7168, 256, 1, 1, True), (4096, 512, 1, 1, True),
    (256, 256, 1, 2, False), (256, 2048, 1, 4, False), (512, 512, 1, 1, False), (1024, 1024, 1, 8, False), (2048, 512, 1, 4, False),
    (7168, 384, 1, 4, False)])
def test_few_tokens_form(ask, d, I, elem, T, stream):
    assert ask([("few", d, I, elem, T)])[0] == (int(stream),)


# widths, bytes of a weight, rows of the layer-step, experts that have any (with equal shares), whether the grouped GEMM is the bf16 one of
# 128-column tiles, and whether streaming beats it
@pytest.mark.parametrize("d,I,elem,rows,used,grouped,stream", [
    (2048, 768, 2, 296, 115, True, True), (2048, 768, 2, 640, 128, True, True), (2048, 768, 2, 705, 128, True, False),
    (2048, 768, 2, 384, 64, True, True), (2048, 768, 2, 512, 64, True, False), (2048, 768, 2, 128, 32, True, True),
    (2048, 768, 2, 256, 32, True, False), (2048, 768, 2, 128, 8, True, False), (2048, 768, 2, 512, 16, True, False),
    (512, 512, 2, 256, 128, True, False), (512, 512, 2, 640, 128, True, False), (256, 128, 2, 64, 16, True, False),
    (1024, 1024, 2, 384, 128, True, True), (1024, 1024, 2, 512, 128, True, False), (1024, 2816, 2, 256, 64, True, True),
    (1024, 2816, 2, 320, 64, True, False), (1024, 2816, 2, 80, 16, True, True), (1024, 2816, 2, 128, 16, True, False),
    (768, 768, 2, 640, 128, True, True), (3072, 1024, 2, 192, 64, True, True), (3072, 1024, 2, 320, 64, True, False),
    (4096, 14336, 2, 40, 8, True, True), (4096, 14336, 2, 48, 8, True, False), (4096, 14336, 2, 32, 2, True, False),
    (4096, 14336, 2, 96, 16, True, False), (5120, 8192, 2, 64, 16, True, True), (5120, 8192, 2, 80, 16, True, False),
    (1472, 704, 2, 280, 61, False, True), (1472, 704, 2, 366, 61, False, False), (320, 192, 2, 60, 60, False, False),
    (7168, 2048, 1, 128, 64, False, False)])
def test_token_batch_form(ask, d, I, elem, rows, used, grouped, stream):
    items = used * -(-rows // (8 * used))
    assert ask([("batch", d, I, elem, rows, used, items, used * I // 128 if grouped else 0)])[0] == (int(stream),)


def test_token_batch_form_counts_second_reads(ask):
    # 640 rows of 128 experts stream while none has more than eight; with 60 experts read twice they do not
    assert ask([("batch", 2048, 768, 2, 640, 128, i, 768) for i in (128, 188)]) == [(1,), (0,)]
