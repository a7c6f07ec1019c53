// Launch plans of the library's host code, one request per line of stdin:
//   height MODEL A B C N ORDER ROWS GROUPS SWEEPS WANTED
// prints the plan "S TR TG HR HG tiles lds" (LDS bytes), or "refused".
//   height_auto MODEL A B C N ORDER ONE_BIT
// prints the automatic shape "TR TG S" and the granules of its tiles.
//   domino_auto N ORDER WEIGHTED T0 SWEEPS
// prints the automatic shape "TR TG S", and of that many sweeps from sweep T0 on
// how many take it.
//   batch ONE_BIT METROPOLIS TASKS THREADS
// prints 1 if a batched chain of that many tasks lists the movable ones.
//   batch_lds STATE_BYTES LISTS THREADS
// prints the static LDS of the batch kernels (with lists or without) and the
// work-groups counted per CU.
#include <cstdio>
#include <cstring>

#include "internal.hpp"

int main()
{
    char line[256], what[32];
    while (std::fgets(line, sizeof line, stdin)) {
        int at = 0;
        if (std::sscanf(line, "%31s%n", what, &at) != 1) continue;
        if (!std::strcmp(what, "height")) {
            tl::HeightDev d{};
            tl::HeightTile t;
            unsigned wanted = 0;
            if (std::sscanf(line + at, "%d %d %d %d %d %u %u %u %u %u", &d.model, &d.a, &d.b, &d.c, &d.N, &t.order,
                            &t.TR, &t.TG, &t.S, &wanted) != 10)
                return 1;
            (void)tl::height_words(d);
            tl::TilePlan p;
            if (tl::height_plan(d, t, wanted, &p))
                std::printf("%u %u %u %u %u %u %u\n", p.S, p.TR, p.TG, p.HR, p.HG, p.tiles(), p.lds);
            else
                std::printf("refused\n");
        } else if (!std::strcmp(what, "height_auto")) {
            tl::HeightDev d{};
            unsigned order, one_bit;
            if (std::sscanf(line + at, "%d %d %d %d %d %u %u", &d.model, &d.a, &d.b, &d.c, &d.N, &order, &one_bit) != 7)
                return 1;
            (void)tl::height_words(d);
            tl::HeightTile t = tl::height_auto_tile(d, one_bit != 0, order != 0);
            t.order = order;
            tl::TilePlan p;
            if (!tl::height_plan(d, t, 1u << 20, &p)) return 1;
            std::printf("%u %u %u %u\n", t.TR, t.TG, t.S,
                        tl::height_lds(d.model != TL_LOZENGE, p.TR + 2u * p.HR, p.TG + 2u * p.HG).granules);
        } else if (!std::strcmp(what, "domino_auto")) {
            tl::DominoDev d{};
            unsigned order, weighted, t0, sweeps;
            if (std::sscanf(line + at, "%d %u %u %u %u", &d.n, &order, &weighted, &t0, &sweeps) != 5) return 1;
            (void)tl::domino_words(d.n, &d.ng, &d.RS, &d.PS);
            tl::DominoTile t = tl::domino_auto_tile(d.n, order != 0, weighted != 0), late;
            t.order = order;
            const unsigned early = weighted ? sweeps : tl::domino_spread(d, t, t0, sweeps, &late);
            std::printf("%u %u %u %u", t.TR, t.TG, t.S, early);
            if (early < sweeps) std::printf(" %u %u %u", late.TR, late.TG, late.S);
            std::printf("\n");
        } else if (!std::strcmp(what, "batch")) {
            unsigned one_bit, metro, tasks, threads;
            if (std::sscanf(line + at, "%u %u %u %u", &one_bit, &metro, &tasks, &threads) != 4) return 1;
            std::printf("%d\n", tl::batch_lists(one_bit != 0, metro != 0, tasks, threads) ? 1 : 0);
        } else if (!std::strcmp(what, "batch_lds")) {
            unsigned state, lists, threads;
            if (std::sscanf(line + at, "%u %u %u", &state, &lists, &threads) != 3) return 1;
            std::printf("%u %u\n", tl::batch_static_lds(lists != 0), tl::batch_per_cu(state, lists != 0, threads));
        } else {
            return 1;
        }
    }
    return 0;
}
