"""Host-side logic of bench.py (CPU): the code digest that keys the committed
HBM-traffic summaries to the kernel sources they were measured on."""
import os
import re
import shutil

import bench
from paper_2601_05296_amd import synth


def test_code_tokens_drop_comments_only():
    src = ('int a = 1; // a comment\n/* block\n comment */ const char* s = "//kept /*kept*/";\n'
           "char q = '\\''; char r = '/';  int   b;")
    assert bench.code_tokens(src) == ('int a = 1; const char* s = "//kept /*kept*/"; '
                                      "char q = '\\''; char r = '/'; int b;")


def test_digest_ignores_comments_but_not_code(tmp_path):
    d = tmp_path / "csrc"
    shutil.copytree(bench.CSRC, d, ignore=shutil.ignore_patterns("*.o", "*.so"))
    base = bench.source_digest(str(d))
    assert base == bench.source_digest()
    f = d / "ffn.hip"
    text = f.read_text()
    f.write_text("// an added comment line\n" + text.replace("\n", "\n\n", 3))
    assert bench.source_digest(str(d)) == base
    f.write_text(text.replace("RASTER_GM", "RASTER_GM + 0", 1))
    assert bench.source_digest(str(d)) != base



def test_every_launched_kernel_has_a_work_model():
    """bench.kernel_model knows each name the library's probe records (the float32
    GEMMs have no peak here; two kernels move nothing worth counting)."""
    names = set()
    for fn in os.listdir(bench.CSRC):
        if fn.endswith(".hip"):
            for line in open(os.path.join(bench.CSRC, fn)):
                for call in re.findall(r"probe::mark\((.*)", line) + re.findall(r'"sk_g\w+".*', line):
                    names |= set(re.findall(r'"(\w+)"', call))
    assert {"sk_g1", "sk_g2h", "g3h_narrow", "route_pick", "rb_dx", "index_one"} <= names
    cfg = synth.CONFIGS["mid_e64k6"]
    for n in sorted(names):
        amount, unit, bound = bench.kernel_model(n, cfg, 2)
        if n.startswith("f32_g") or n in ("tile_scan", "rb_dwg_reduce"):
            assert amount == 0, n
        else:
            assert amount > 0, n


def test_small_row_gemms_are_priced_by_their_bound():
    """Few rows per expert: the weights read once; many: the products."""
    few = synth.MoEConfig("few", T=48, d=2048, f=1408, E=64, k=6, dtype="bf16", renorm=True)
    amount, unit, bound = bench.kernel_model("sk_g1", few, 2)
    weights = 64 * (1 - (1 - 6 / 64) ** 48) * 2 * 2048 * 1408 * 2
    assert (unit, bound) == ("GB/s", "hbm") and weights < amount < 1.02 * weights
    many = synth.CONFIGS["mid_e64k6"]
    assert bench.kernel_model("sk_g1", many, 2) == bench.kernel_model("g1_kernel", many, 2)


def test_kernel_short_names():
    """Profiler names without namespaces, parameters and template arguments, also
    where an argument is a type of the namespace."""
    ns = "moe::(anonymous namespace)::"
    for full, short in (
            ("void %sg5_kernel<0, moe::rs::Cfg<256, 128, 2, 4, 2>, false>(unsigned short const*, int)" % ns, "g5_kernel"),
            ("void %sg5_kernel<0, moe::rs::Cfg<128, 64, 2, 2, 2>, true>(float*)" % ns, "g5_narrow"),
            ("void %sg2h_kernel<1, true, moe::rs::Cfg<64, 512, 1, 8, 1> >(int)" % ns, "g2h_narrow"),
            ("void %sg3h_kernel<0, moe::rs::Cfg<128, 512, 2, 4, 1>, false>(int)" % ns, "g3h_kernel"),
            ("void %ssk_g2<0, true, false, %sSk<32, 2> >(unsigned short const*, long)" % (ns, ns), "sk_g2"),
            ("%sroute_pick(float const*, long)" % ns, "route_pick"),
            ("__amd_rocclr_copyBuffer", "__amd_rocclr_copyBuffer"),
            ("void at::native::vectorized_elementwise_kernel<4, at::native::FillFunctor<float>, "
             "std::array<char*, 1ul> >(int, at::native::FillFunctor<float>)", "vectorized_elementwise_kernel")):
        assert bench.kernel_short_name(full) == short, full
