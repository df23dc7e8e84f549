"""The dispatch rules by themselves (CPU): the GPU tests' cases reach the forms that they name, and
no sizes ask for a form that is not compiled."""
import itertools

from _shapes import CUS, ROUTE_FORMS, STREAM_FORMS, SUMS_FORMS, TILE_FORMS, WIDE_FORMS, ask, empty_beside


def _route(dtype, T, h, E, k, want=1):
    return f"route {int(dtype == 'bf16')} {T} {h} {E} {k} {want} {CUS}"


def test_route_cases_reach_their_forms():
    got = ask([_route(*c[:5]) for c in ROUTE_FORMS])
    assert got == [c[5] for c in ROUTE_FORMS]


def test_every_route_form_is_compiled():
    # (blocks, steps) per number of experts, as route.hip compiles them
    built = {16: {"1 x 4", "1 x 6", "2 x 2", "2 x 3", "4 x 2"}, 32: {"1 x 2", "1 x 5", "2 x 1", "4 x 1"}, 64: {"1 x 3", "2 x 1", "4 x 1"},
             128: {"1 x 1", "2 x 1"}, 256: {"1 x 1", "2 x 1"}}
    sizes = list(itertools.product(("bf16", "f32"), (1, 16, 17, 32, 33, 64, 65, 4096, 4097, 16383, 16384, 100000),
                                   (8, 64, 256, 328, 512, 768, 1024, 1032, 2048, 4096), (1, 16, 17, 32, 33, 64, 65, 128, 129, 256),
                                   (1, 8, 9), (0, 1)))
    got = ask([_route(d, T, h, E, min(k, E), want) for d, T, h, E, k, want in sizes])
    for (d, T, h, E, k, want), form in zip(sizes, got):
        if form.startswith("lds"):
            continue
        n = next(v for v in built if E <= v)
        assert form.removesuffix(" grouped") in built[n], (d, T, h, E, k, want, form)
        if form.endswith(" grouped"):
            assert T <= 16 * int(form.split()[0]) and min(k, E) <= 8 and want


def test_the_kernel_of_a_token_does_not_depend_on_its_batch():
    # the two routing kernels sum K in different orders: which one is a matter of type, h and E
    for d, h, E in itertools.product(("bf16", "f32"), (64, 72, 4096), (1, 24, 32, 33, 64, 256)):
        got = ask([_route(d, T, h, E, 1) for T in (1, 16, 17, 64, 65, 8192, 100000)])
        assert len({g.startswith("lds") for g in got}) == 1


def _ffn(A, E, h, f, act, dtype="bf16"):
    return f"ffn {int(dtype == 'bf16')} {A} {E} {h} {f} {int(act == 'swiglu')} {CUS}"


def test_expert_step_cases_reach_their_forms():
    cases = [(sum(c), len(c), h, f, act, form) for c, h, f, act, form in TILE_FORMS + STREAM_FORMS]
    cases += [(A, E, h, f, act, form) for E, A, h, f, act, form in SUMS_FORMS]
    for c, h, f, forms, beside in WIDE_FORMS:
        A, E = sum(c), len(c)
        cases += [(A, E, h, f, act, form) for act, form in forms.items()]
        cases += [(A, E + empty_beside(A, E), h, f, act, form) for act, form in beside.items()]
    got = ask([_ffn(*c[:5]) for c in cases])
    assert got == [c[5] for c in cases]


def test_weights_stream_only_where_re_reading_them_pays():
    # (rows, experts, h, f, act): measured faster streamed, and faster in tiles
    streamed = [(128, 1, 4096, 3584, "swiglu"), (512, 1, 2048, 2048, "gelu"), (384, 8, 2048, 2048, "gelu"),
                (512, 16, 1024, 4096, "gelu"), (512, 8, 1024, 4096, "gelu"), (512, 24, 1032, 4096, "gelu"),
                (1024, 64, 1024, 1024, "gelu"), (192, 4, 4096, 1792, "swiglu")]
    tiled = [(512, 1, 4096, 3584, "swiglu"), (512, 8, 4096, 3584, "swiglu"), (384, 2, 4096, 3584, "swiglu"),
             (256, 8, 4096, 3584, "swiglu"), (512, 8, 4096, 1792, "swiglu")]
    assert all(a.startswith("stream") for a in ask([_ffn(*c) for c in streamed]))
    assert not any(a.startswith("stream") for a in ask([_ffn(*c) for c in tiled]))


def test_few_tiles_take_small_ones():
    # a long K and rows enough per expert for 256 x 256 tiles, but too few of them for the CUs
    got = ask([_ffn(768, 1, 1024, 4096, "gelu"), _ffn(1536, 8, 1024, 4096, "gelu"), _ffn(6144, 16, 1024, 4096, "gelu"),
               _ffn(8192, 16, 1024, 4096, "gelu"), _ffn(3008, 64, 1024, 1024, "gelu"), _ffn(3008, 64, 768, 768, "gelu")])
    assert [a.split(" / ")[1] for a in got] == ["128x128", "128x128", "128x256", "turns", "128x256", "64x256"]


def test_wide_tiles_that_may_not_fit_one_round():
    # up-projection: tiles that fit one round of the CUs in any likely routing, and that may not
    up = ask([_ffn(A, E, h, f, "swiglu") for A, E, h, f in
              [(2048, 2, 4096, 3584), (4096, 2, 4096, 1792), (3072, 8, 4096, 1792),
               (4096, 4, 4096, 1792), (2429, 3, 6144, 2816), (3847, 16, 4096, 1408)]])
    assert [a.split(" / ")[0] for a in up] == ["turns"] * 3 + ["pairs"] * 3
    # down-projection: 128-row tiles that fit one round of two a CU where 256-row ones may not fit theirs
    down = ask([_ffn(A, E, h, f, "gelu") for A, E, h, f in
                [(4674, 8, 3072, 2816), (5170, 2, 3072, 3072), (3674, 12, 3072, 3072), (18538, 32, 768, 3072),
                 (16384, 4, 1024, 4096), (8192, 16, 1024, 4096)]])
    assert [a.split(" / ")[1] for a in down] == ["128x256"] * 4 + ["turns"] * 2
