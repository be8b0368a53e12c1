// Replay of the factorisation's schedule (csrc/qqq_factor_schedule.h) without its arithmetic: `slots` of `grid` workgroups are resident, each
// moves at random; a step of one is a draw, a wait that is over, or a task's end.  Every tile has to receive every panel once and in order, and all
// waits have to end.  usage: factor_replay nb grid slots help seed -> exit code 0: done, 1: nobody can move, 2: a task ran too early or twice
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "qqq_factor_schedule.h"

using namespace qqq;

int main(int argc, char** argv) {
  if (argc != 6) return 3;
  const int nb = atoi(argv[1]), grid = atoi(argv[2]), slots = atoi(argv[3]);
  const bool help = atoi(argv[4]) != 0;
  std::mt19937 rng(atoi(argv[5]));
  const Flags f = {nb};
  std::vector<int> flag(nb + 2 * nb * nb, 0), panels(nb * nb, 0), solved(nb * nb, 0), factored(nb, 0);  // what was told, and what was done
  int arrived = 0, drawn[3] = {0, 0, 0}, ended = 0;
  enum State { kDraw, kWait, kWork };
  struct Group { int number; State state; Queue queue; Task task; int k; bool half, owes; };  // the last three: the chain's
  std::vector<Group> here;
  auto bad = [&](const char* what, const Task& t) { printf("%s: kind %d tile (%d, %d) panels %d + %d\n", what, t.kind, t.i, t.j, t.p0, t.np); exit(2); };
  auto holds = [&](const Need& n) { return !n.asks || flag[n.flag] >= n.least; };
  auto ready = [&](const Task& t) { for (int l = 0; l < 64; ++l) if (!holds(need_of(f, t, l))) return false; return true; };
  auto receive = [&](int i, int j, int p0, int np, const Task& t) {  // panels from the last down, each once
    if (i > j) return;
    for (int p = p0 + np - 1; p >= p0; --p) {
      if (panels[i * nb + j] != nb - 1 - p || !solved[p * nb + i] || !solved[p * nb + j]) bad("update", t);
      panels[i * nb + j] = nb - p;
    }
  };
  auto solve = [&](int i, int k, const Task& t) {
    if (!factored[k] || solved[k * nb + i] || panels[i * nb + k] != nb - k - 1) bad("solve", t);
    solved[k * nb + i] = 1;
  };
  auto finish = [&](const Task& t) {
    if (t.kind == kSolve) solve(t.i, t.j, t);
    if (t.kind == kUpdate64) receive(t.i, t.j, t.p0, t.np, t);
    if (t.kind == kUpdate128) for (int x = 0; x < 4; ++x) receive(t.i + x / 2, t.j + x % 2, t.p0, t.np, t);
    for (int l = 0; l < 64; ++l) {
      const Done d = done_of(f, t, l);
      if (d.tells) flag[d.flag] = d.value;
    }
  };
  // one move of a group; false: it has to wait.  2: it is through
  auto move = [&](Group& g) -> int {
    if (g.state == kWait) {
      if (!ready(g.task)) return 0;
      g.state = kWork;
      return 1;
    }
    if (g.state == kWork) {
      finish(g.task);
      g.state = kDraw;
      return 1;
    }
    if (g.number == 0) {
      if (holds(need_of_chain(f, g.k, g.half))) {
        const Task own = {kNothing, g.k, g.k, 0, 0};
        if (!g.half) {
          if (g.k + 1 < nb) {
            flag[f.solved(g.k + 1, g.k)] = 1;
            receive(g.k, g.k, g.k + 1, 1, own);
          }
          if (panels[g.k * nb + g.k] != nb - 1 - g.k) bad("factor", own);
          factored[g.k] = 1;
          g.half = true;
          return g.k == 0 ? 2 : 1;
        }
        flag[f.factored(g.k)] = 1;
        solve(g.k - 1, g.k, own);
        g.half = false;
        --g.k;
        return 1;
      }
      if (!help || arrived >= kFactorCrew) return 0;
      if (g.half) flag[f.factored(g.k)] = 1;  // what it owes the others
      else flag[f.solved(g.k + 1, g.k)] = 1;
      const int q = queue_for_chain(nb, g.k, drawn[1], drawn[2], &g.queue);
      if (q == 0) return 0;
      g.task = task_of(g.queue.step, q, drawn[q]++ - g.queue.base);
      g.state = g.task.kind == kNothing ? kDraw : kWait;
      return 1;
    }
    const int ticket = drawn[g.queue.queue]++;
    if (!g.queue.reach(ticket)) {
      if (g.queue.queue == 1) return 2;
      g.queue = Queue(1, nb);
      return 1;
    }
    g.task = task_of(g.queue.step, g.queue.queue, ticket - g.queue.base);
    g.state = g.task.kind == kNothing ? kDraw : kWait;
    return 1;
  };
  while (ended < grid) {
    std::vector<int> order;
    if ((int)here.size() < slots && arrived < grid && (here.empty() || rng() % 3 == 0)) {
      const int number = arrived++;
      here.push_back({number, kDraw, Queue(number % 3 == 1 ? 1 : 2, nb), {}, nb - 1, false, false});
    }
    for (int i = 0; i < (int)here.size(); ++i) order.push_back(i);
    std::shuffle(order.begin(), order.end(), rng);
    int moved = 0;
    for (int i : order) {
      moved = move(here[i]);
      if (moved) {
        if (moved == 2) here.erase(here.begin() + i), ++ended;
        break;
      }
    }
    if (!moved) {
      if ((int)here.size() < slots && arrived < grid) continue;  // another one may come
      printf("nobody can move: %d resident\n", (int)here.size());
      return 1;
    }
  }
  for (int k = 0; k < nb; ++k)
    if (!factored[k]) return 2;
  return 0;
}
