"""Chunk lengths of a solve and the places of its kept graphs (host rules)."""
import pytest

from tests.host_harness import run_cpp


def test_graphs_are_replaced_only_when_nothing_runs(tmp_path):
    """A handle solves with check_every 3, then 5, then the default: the two
    chunk lengths, launched without a wait in between, keep places of their
    own, whatever other lengths came before."""
    out = run_cpp(tmp_path, ["pace.h"], r"""
    int32_t held[kGraphs] = {};
    int captured = 0, replaced_running = 0;
    bool running[kGraphs] = {};
    auto launch = [&](int32_t n) {
        const int g = graph_place(n);
        if (held[g] != n) {
            replaced_running += held[g] && running[g];
            held[g] = n;
            ++captured;
        }
        running[g] = true;
    };
    auto look = [&] { for (bool &r : running) r = false; };
    for (int32_t every : {3, 5, 3})
        for (int i = 0; i < 4; ++i) { launch(every); look(); }
    for (int i = 0; i < 6; ++i) {
        launch(kLongChunk);
        launch(kChunk);
        launch(kChunk);
        look();
    }
    std::printf("%d %d\n", captured, replaced_running);
""")
    assert out == ["5", "0"]      # 3, 5, 3, then 16 and 4 once each


@pytest.mark.parametrize("every", [32, 128])
def test_chunks_follow_the_rate(tmp_path, every):
    """|r|^2 falls a hundredfold every ten iterations: the looks come no later
    than every check_every iterations and hit the end within a chunk."""
    out = run_cpp(tmp_path, ["pace.h"], r"""
    struct State { double rr, tol2; int32_t iter, status; } s{1.0, 1e-16, 0, 0};
    Pace p;
    p.every = %d;
    int looks = 0;
    while (s.rr > s.tol2 && looks < 1000) {
        const int32_t n = p.next(&s, 1, 0);
        if (n < 1 || n > p.every) return 1;
        s.iter += n;
        s.rr = std::pow(10.0, -0.2 * s.iter);
        ++looks;
    }
    std::printf("%%d %%d\n", s.iter, looks);
""" % every)
    it, looks = map(int, out)
    assert 80 <= it < 84 and looks <= 8


def test_tolerance_that_underflows(tmp_path):
    """rtol |b| whose square is zero is never met: looks every check_every
    iterations, as for any solve that is far from its end."""
    out = run_cpp(tmp_path, ["pace.h"], r"""
    struct State { double rr, tol2; int32_t iter, status; } s{1.0, 0.0, 0, 0};
    Pace p;
    for (int i = 0; i < 5; ++i) {
        const int32_t n = p.next(&s, 1, 0);
        s.iter += n;
        s.rr *= 1e-3;
        std::printf("%d ", n);
    }
""")
    assert out == ["32"] * 5
