// The order of the work of factor_kernel (qqq_compensate.hip), for the kernel and for a replay on the host: which tasks there are, what each
// waits for and what it tells the others.
//
// H = R D R^T in blocks of 64 channels from the last, nb of them.  The chain (one workgroup) factors block k, solves tile k - 1 of panel k and takes that
// off the tile that it factors next.  The other workgroups draw tickets of two queues for the rest; all tasks have one order (step by step from the
// last block, in a step queue 2 before queue 1), in which a task needs only earlier ones and the chain's blocks k and after.
#ifndef QQQ_FACTOR_SCHEDULE_H_
#define QQQ_FACTOR_SCHEDULE_H_

#ifdef __HIPCC__
#include <hip/hip_runtime.h>
#define QQQ_SCHEDULE __host__ __device__ __forceinline__
#else
#define QQQ_SCHEDULE inline
#endif

namespace qqq {

constexpr int kOuter = 4;  // blocks whose columns receive panels together
// Workgroups that keep chain and queues going: the chain and one on each queue.  While fewer have come, the chain takes tasks where it would wait.
constexpr int kFactorCrew = 3;

QQQ_SCHEDULE int schedule_min(int a, int b) { return a < b ? a : b; }
QQQ_SCHEDULE int schedule_max(int a, int b) { return a > b ? a : b; }
QQQ_SCHEDULE int triangle(int n) { return n * (n + 1) / 2; }

// The tasks of one step (block k).  Queue 2: far updates, i.e. by the four panels after block k's four, of the four blocks before
// these (whose turn comes next), then a quarter of the others.  Queue 1: the solves of panel k, its updates of its own four blocks and, every
// second step, those of the four before by two panels.
struct Tasks {
  int k, g, nb, p0, np;  // g: block k's four; panels [p0, p0 + np) of the four after
  int n_next, far0, n_far, n_solve, n_near, n_pair;
  QQQ_SCHEDULE Tasks(int nb_, int k_) : k(k_), g(k_ / kOuter), nb(nb_) {
    p0 = kOuter * (g + 1);
    np = p0 < nb ? schedule_min(kOuter, nb - p0) : 0;
    const int own = kOuter * g, n = schedule_max(own - kOuter, 0), wide = triangle(n / 2), quarter = p0 - 1 - k;
    n_next = np && k == p0 - 1 && g > 0 ? triangle(own) - triangle(n) : 0;
    far0 = np ? wide * quarter / kOuter : 0;
    n_far = np ? wide * (quarter + 1) / kOuter - far0 : 0;
    n_solve = schedule_max(k - 1, 0);
    n_near = k > own ? triangle(k) - triangle(own) - 1 : 0;
    n_pair = g > 0 && (k == own || (k == own + 1 && own + 2 < nb)) ? triangle(own) - triangle(n) : 0;
  }
  QQQ_SCHEDULE int count(int queue) const { return queue == 1 ? n_solve + n_near + n_pair : n_next + n_far; }
};

// A queue as it is drawn from: the step that a ticket belongs to.
struct Queue {
  int queue, base;  // the tickets of earlier steps
  Tasks step;
  QQQ_SCHEDULE Queue(int queue_, int nb) : queue(queue_), base(0), step(nb, nb - 1) {}
  QQQ_SCHEDULE bool reach(int ticket) {  // false: there is no such task
    while (ticket - base >= step.count(queue) && step.k > 0) {
      base += step.count(queue);
      step = Tasks(step.nb, step.k - 1);
    }
    return ticket - base < step.count(queue);
  }
};

struct Tile64 { int i, j; };
// tile number u of a triangle counted from its last: columns from the last, rows from the diagonal up
QQQ_SCHEDULE Tile64 tile_from_last(int total, int u) {
  const int v = total - 1 - u;
  int j = (int)((__builtin_sqrtf(8.0f * (float)v + 1.0f) - 1.0f) * 0.5f);  // column j starts at j (j + 1) / 2
  while (j * (j + 1) / 2 > v) --j;
  while ((j + 1) * (j + 2) / 2 <= v) ++j;
  return {v - j * (j + 1) / 2, j};
}

// A task: the solve of tile i of panel j; or what tile (i, j) receives from panels [p0, p0 + np), as one tile of 64 x 64 or
// with those at (i + 1, j), (i, j + 1), (i + 1, j + 1) as one of 128 x 128 (below the diagonal there is nothing).
enum TaskKind { kNothing, kSolve, kUpdate64, kUpdate128 };
struct Task { TaskKind kind; int i, j, p0, np; };
QQQ_SCHEDULE Task task_of(const Tasks& s, int queue, int at) {
  if (queue == 1) {
    const int near = at - s.n_solve, pair = near - s.n_near, own = kOuter * s.g;
    if (near < 0) return {kSolve, s.k - 2 - at, s.k, 0, 0};
    if (pair < 0) {
      const Tile64 t = tile_from_last(triangle(s.k), near + 1);  // (the first is the chain's)
      return {kUpdate64, t.i, t.j, s.k, 1};
    }
    const Tile64 t = tile_from_last(triangle(own), pair);
    int p0 = own + (s.k == own ? 0 : 2), np = schedule_min(2, s.nb - p0);
    if (s.k == own && pair == 0) ++p0, --np;  // (the chain takes panel k off the tile that it factors next)
    return {np > 0 ? kUpdate64 : kNothing, t.i, t.j, p0, np};
  }
  if (at < s.n_next) {
    const Tile64 t = tile_from_last(triangle(kOuter * s.g), at);
    return {kUpdate64, t.i, t.j, s.p0, s.np};
  }
  const Tile64 t = tile_from_last(triangle(kOuter / 2 * (s.g - 1)), at - s.n_next + s.far0);
  return {kUpdate128, 2 * t.i, 2 * t.j, s.p0, s.np};
}

// Flags, one array: blocks factored, [nb]; panels that tile (i, j) has received, [nb][nb]; tile i of panel k solved, at [k][i], [nb][nb].
struct Flags {
  int nb;
  QQQ_SCHEDULE int factored(int k) const { return k; }
  QQQ_SCHEDULE int applied(int i, int j) const { return nb + i * nb + j; }
  QQQ_SCHEDULE int solved(int k, int i) const { return nb + nb * nb + k * nb + i; }
};

// What lane `lane` of 64 waits for before a task: flags[flag] >= least, if it asks
struct Need { int flag, least; bool asks; };
QQQ_SCHEDULE Need need_of(const Flags& f, const Task& t, int lane) {
  const int nb = f.nb;
  if (t.kind == kSolve) return {lane == 0 ? f.factored(t.j) : f.applied(t.i, t.j), lane == 0 ? 1 : nb - t.j - 1, lane < 2};
  const int panel = schedule_min(t.p0 + (lane & 3), nb - 1);
  if (t.kind == kUpdate64)  // lanes 0 .. 3 and 4 .. 7: the panels' tiles i and j; lane 8: the tile itself
    return {lane < 8 ? f.solved(panel, lane < 4 ? t.i : t.j) : f.applied(t.i, t.j), lane < 8 ? 1 : nb - t.p0 - t.np, lane < 8 ? (lane & 3) < t.np : lane == 8};
  // lanes 0 .. 15: row tiles i, i + 1, j, j + 1 of the panels; lanes 16 .. 19: the four tiles themselves, the one below the diagonal left out
  const int ti = t.i + ((lane >> 1) & 1), tj = t.j + (lane & 1), tile = lane >> 2;
  return {lane < 16 ? f.solved(panel, (tile < 2 ? t.i : t.j) + (tile & 1)) : f.applied(ti, tj), lane < 16 ? 1 : nb - t.p0 - t.np,
          lane < 16 ? (lane & 3) < t.np : lane < 20 && ti <= tj};
}
// What a task tells when it is done: flags[flag] = value, of lane 0, and for a tile of 128 x 128 of lanes 0 .. 3, where it tells
struct Done { int flag, value; bool tells; };
QQQ_SCHEDULE Done done_of(const Flags& f, const Task& t, int lane) {
  if (t.kind == kSolve) return {f.solved(t.j, t.i), 1, lane == 0};
  if (t.kind == kUpdate64) return {f.applied(t.i, t.j), f.nb - t.p0, lane == 0};
  const int ti = t.i + ((lane >> 1) & 1), tj = t.j + (lane & 1);
  return {f.applied(ti, tj), f.nb - t.p0, lane < 4 && ti <= tj};
}

// The chain's waits at block k: before the block's tile is loaded, and, the block factored, before row tile k - 1 is
QQQ_SCHEDULE Need need_of_chain(const Flags& f, int k, bool factored) {
  if (factored) return {f.applied(k - 1, k), f.nb - k - 1, true};
  return {f.applied(k, k), schedule_max(f.nb - k - 2, 0), true};
}

// The queue whose next task the chain takes on where it would wait at block k, `drawn` tickets of queues 1 and 2 being gone; 0: none.  It is the first in
// the order of all that nobody has drawn, so what it needs is done or in the hands of workgroups whose own tasks come earlier still; and its step
// is one that the chain has done with, so it needs nothing more of the chain.
QQQ_SCHEDULE int queue_for_chain(int nb, int k, int drawn1, int drawn2, Queue* head) {
  Queue one(1, nb), two(2, nb);
  const bool any1 = one.reach(drawn1), any2 = two.reach(drawn2);
  const bool second = any2 && (!any1 || two.step.k >= one.step.k);
  if (!any1 && !any2) return 0;
  *head = second ? two : one;
  return head->step.k > k ? head->queue : 0;
}

}  // namespace qqq

#endif  // QQQ_FACTOR_SCHEDULE_H_
